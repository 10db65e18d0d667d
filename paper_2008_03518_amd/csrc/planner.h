// planner.h -- device-side data layout shared by the HIP translation units of
// libfastmdp (internal; the public boundary is include/fastmdp.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fastmdp.h"

namespace fmdp {

constexpr int kPlanThreads = 1024;  // planning workgroup: one request per CU, 16 wave64
constexpr int kPairThreads = 512;   // full sweep of more requests than CUs: two per CU, 8 wave64 each
constexpr int kPairTile = 2048;     // row entries they stage at a time (two workgroups share a CU's LDS)
constexpr int kPairHeads = 64;      // headings up to which a pair's workgroup has eight slices
constexpr int kPropThreads = 512;   // with the proposal path: 8 wave64, twice the registers per lane
constexpr int kRangeThreads = 256;  // range-query planner: 4 wave64, up to four requests per CU
constexpr int kRangePerCU = 4;      // range-query workgroups resident per CU (LDS and registers)
constexpr int kLaunchPerCU = 2;     // FCFS requests per CU in a launch (no proposal, no window)
constexpr int kRangeThreadsSolo = 512;  // range-query planner alone on a CU: 8 wave64, one action per thread
constexpr int kRangeMaxHeads = 64;  // headings the range-query planner takes (its LDS budget)
constexpr int kMaxActions = 512;
constexpr int kMaxPoints = 4 * 4096;  // trajectory points per request (max_steps + 1)
constexpr int kMaxHeads = 128;
constexpr int kMaxLookahead = 16;   // longest scoring window W (steps)
constexpr int kRunning = -1;        // slot status while a request is being planned
constexpr int kAlive = 0x7fffffff;  // table entry death epoch of a live entry
constexpr double kBand = 1e-3;      // metres: FP32 nearest distances this close to the well
                                    // radius are recomputed exactly in FP64

// Problem constants as the kernels use them (passed by value).
struct DevCfg {
    double box_lo[3], box_hi[3];
    double dt, ell;
    double gamma, r_goal, r_intr, R_intr, gamma_intr, R_sep, r_terr, R_terr, gamma_terr;
    double log_gamma, log_gamma_intr, log_gamma_terr;   // discounts as exp(log_gamma * distance/ell)
    double abs_r_goal, abs_r_intr, abs_r_terr;
    float log2_gamma_f, inv_ell_f, abs_r_goal_f;        // FP32 goal-term bound of the proposal
    double climb[FASTMDP_MAX_ACT_DIM], speed[FASTMDP_MAX_ACT_DIM];
    float kv[FASTMDP_MAX_ACT_DIM];       // -2 * speed * dt
    float climb_f[FASTMDP_MAX_ACT_DIM];  // climb rates
    float zeta_scale;                    // -2 * dt
    double tie_rel;
    double reach;                        // max(R_intr, R_sep) + 1 m: a plan farther than this from
                                         // a successor cannot change its value
    double band_lo2, band_hi2;           // (R_intr -+ kBand)^2: squared distances recomputed exactly
    double reach_state;                  // reach + longest action step: a plan farther than this
                                         // from a state cannot change any of its successors' values
    int n_head, n_climb, n_speed, n_actions;
    int zero_climb;                      // index of the zero climb rate in the middle, else -1
    int max_steps;
    int lookahead;                       // scoring window W >= 1 (Alg. 1 forward projections)
    int range_query;                     // 1: stage only the row entries within cull_r2 of the state
    float cull_r2;                       // squared staging radius of the range query (FP32, 1 m margin)
    double max_step;                     // longest action step [m]: window point w lies within
                                         // w * max_step of the state
    double peak_growth;                  // co-simulated batch: peak radius R_intr + peak_growth * tau
    float cull_box;                      // half-width of the range-query box test on x and y: the
                                         // staging radius plus a margin for every rounding of the
                                         // exact test (FP32 offsets of coordinates up to max_abs)
    // runs of steps that no plan affects (range.hip): the goal-directed
    // action is the choice when every other action's successor is farther
    // from the goal by more than run_margin, while the goal is within
    // run_dmax; run_v is the fastest speed, run_c1 the largest cosine of the
    // other headings' offsets, run_ok 0 where the goal term does not decide
    // (no goal reward, a wide tie band) or the box test's half-widths run_r
    // (in steps of the table's 16-bit x | y << 16) do not fit
    double run_margin, run_dmax, run_c1;
    uint32_t run_r, run_w, run_step;     // run_w: the box's widths (everything where they do not fit);
                                         // run_step: the longest action step in the same units
    int run_v, run_ok;
    int detour_ok;                       // an action inside a well never beats one outside every well
    double clear_terr;                   // terrain clearance of a step that the goal term decides: clear of
                                         // the terrain well, and not below the surface (max(R_terr, 0))
    int longest_row;                     // entries of the longest row when the call began (uses_pairs)
    int planner_threads;                 // full-sweep path: 0 (automatic), kRangeThreads, kRangeThreadsSolo,
                                         // kPlanThreads
    int n_cu;                            // compute units of the device
};

// Time-major structure-of-arrays known-plan table.  Entry j of row t is at
// [t * cap + j] in X, Y, Z, vis, own, dead; rowN[t] entries are in use, in
// append order.  own is the sequence number of the request that owns the
// entry (-1 for loaded plans); dead is the epoch at which a tentative entry
// was withdrawn (kAlive while it stands); vis is own while the entry stands
// and kAlive once withdrawn, so that a request with sequence number q sees
// exactly the entries with vis < q (the planner reads X, Y, Z, vis only).
struct DevTable {
    float *X, *Y, *Z;
    int *vis, *own, *dead;
    // Range-query planner (null without): 16-bit box coordinates of every
    // entry (x | y << 16, quantised below), and per row the entries before
    // column gn[t] that stand, by cell of a kGrid x kGrid grid over the box:
    // records (x, y, z, visibility bits) of cell c of row t at grec[t * cap +
    // goff[t * (kGrid^2 + 1) + c] ..).  Later columns are searched one by one.
    uint32_t *Q;
    float4 *grec;
    int *goff, *gn;
    float qx0, qy0, qsx, qsy;            // box corner, 16-bit steps per metre
    float gsx, gsy;                      // cells per metre
    int *rowN;
    int cap, rows;
    const float *terr;                   // nullptr without terrain
    int tnx, tny;
    double tx0, ty0, tcell;
};

// One request being planned.
struct Slot {
    double origin[3], goal[3];
    int t0;
    int n_points;     // points already in the trajectory (0 = fresh request)
    int status;       // kRunning or a FASTMDP_* plan status
    int req;          // request index (host bookkeeping)
    long long pairs;  // pair evaluations, accumulated
    long long entries;  // table row entries read (16 bytes each), accumulated
    int steps;        // steps taken, accumulated
    int resume_at;    // FCFS check: first affected point, -1 if none
    int seq;          // sequence number: sees live table entries with own < seq
    int valid;        // OK trajectory passed the commit validation against the entries it saw
    int killed;       // FCFS: withdrew tentative entries in the current pass
    int err;          // FCFS: table or log capacity exceeded
    int cert_hit;     // proposal steps certified, accumulated
    int cert_miss;    // proposal steps that fell back to the full sweep, accumulated
    int first;        // FCFS check: first affected point found so far (INT_MAX if none)
    int resumes;      // FCFS: times the request went back to planning, accumulated
};

// Per-slot trajectory buffers, `stride` points per slot.  seen[k] is the
// number of entries of the row scored to produce point k (for k = 0: the
// departure row of the origin check) and ep[k] the withdrawal epoch up to
// which that scoring is known to be consistent.  top[k] is the action with
// the largest value at that step when the chosen action (the lowest index
// inside the tie band) is not itself the largest, else -1.  col[k] is the
// column of point k's tentative table entry, -1 if none.  nd[k] is the
// nearest-plan squared distance of point k as the step scored it.
struct Traj {
    double *xyz;
    int *act;
    double *val;
    int *seen;
    int *ep;
    int *top;
    int *col;
    double *nd;      // squared distance from point k to the nearest plan of its row, as scored
                     // (infinity for the origin, which the origin check validated exactly)
    int *seenw;      // window W > 1: seenw[k * W + w - 1] is the number of entries of row
                     // t0 + k - 1 + w scored for window point w of the step to point k
    int stride;
};

// Withdrawals of one acceptance pass: every withdrawn piece of a trajectory
// is a segment (first entry, entries, first row, owner) of consecutive rows,
// its entries' column and stored position at first entry + row - first row,
// and its bounding boxes per block of kRowBlock rows (FP32 x min, x max, y
// min, y max) from box seg_box[i] on.
struct DeathLog {
    float *x, *y, *z;
    int *col;
    int4 *seg;
    int *seg_box;
    float4 *box;
    int *n;            // entries, segments, boxes in use
    int cap, seg_cap, box_cap;
};

// Work buffers of the FCFS acceptance pass: the row counts before the
// pass's insertions, the trajectories that entered entries in it (slot,
// first row, points, sequence number), and per slot the bounding box (as
// above) of its points in each block of kRowBlock rows, from the block of
// its first row on; the launch stop counter, cleared for the next launch;
// the host's mirror of the slots (pinned memory).
constexpr int kRowBlock = 64;
constexpr int kRowBlocks = kMaxPoints / kRowBlock + 1;   // row blocks a trajectory can touch
struct PassBufs {
    int *rowN_pre;     // [rows]
    int4 *ins;         // [max_slots]
    int *ins_n;        // [1]
    float4 *box;       // [max_slots * kRowBlocks]
    int *stop;         // [1]
    Slot *mirror;      // [max_slots]
};

// Outputs of a single evaluated step (all device pointers, any may be null).
// feat, logit, topk, cert and pbest are written only with a proposal.
struct EvalOut {
    double *V, *G, *I, *T;
    int *best;
    float *feat, *logit;
    int *topk, *cert, *pbest;
};

// Proposal network weights as the planner reads them: BF16 [out][in]
// (W3 zero-padded to a multiple of 32 rows), FP32 biases.
struct PropNet {
    const uint16_t *W1, *W2, *W3;
    const float *b1, *b2, *b3;
    int n_in, n_hid, n_out;
};

// Proposal selection of a planner launch (mode FASTMDP_PROPOSE_*): the top
// k of the ranking, re-ranked every `refresh` steps and after a fallback.
struct PropArgs {
    int mode, k, refresh;
    PropNet net;
};

constexpr int kGrid = 32;            // cells per side (a query's box covers about two per side of a 30 km box)
constexpr int kGridCells = kGrid * kGrid;
constexpr int kGridMin = 256;        // rows of fewer entries are searched one by one

// Grid cell of a coordinate (clamped to the box; never decreases with it).
__device__ __forceinline__ int grid_cell(float x, float x0, float gs) {
    return (int)fminf(fmaxf((x - x0) * gs, 0.0f), (float)(kGrid - 1));
}

// 16-bit box coordinates of an entry, x | y << 16, clamped to the box: a
// quarter of the bytes of its x and y and one subtraction for both, for a
// box test that leaves a superset of the entries near a state.
__device__ __forceinline__ uint32_t quantised(const DevTable &tb, float x, float y) {
    const float a = fminf(fmaxf((x - tb.qx0) * tb.qsx + 0.5f, 0.0f), 65535.0f);
    const float b = fminf(fmaxf((y - tb.qy0) * tb.qsy + 0.5f, 0.0f), 65535.0f);
    return (uint32_t)a | (uint32_t)b << 16;
}

// Entry j of a row (absolute index idx) is visible to the request with
// sequence number seq.
__device__ __forceinline__ bool entry_visible(const DevTable &tb, size_t idx, int seq) {
    return tb.vis[idx] < seq;
}

// Squared distance, in FP64, between an FP64 point and an FP32 table entry:
// the one separation arithmetic of the planner's exact checks and of commit.
__device__ __forceinline__ double entry_d2(double x, double y, double z, float px, float py, float pz) {
    const double dx = (double)px - x, dy = (double)py - y, dz = (double)pz - z;
    return dx * dx + dy * dy + dz * dz;
}

// Early end of a launch: every workgroup whose request finishes adds one to
// *ctr; once it reaches target the others stop at their next step (they stay
// resumable).  target 0: run the full budget.
struct LaunchStop {
    int *ctr;
    int target;
};

// Peaks of the other aircraft of a co-simulated batch (Sec. V; the peak
// table: five risk wells per aircraft along its extrapolated track): pk[4k ..
// 4k+3] = x, y, z, radius of peak k, owner[k] its aircraft's slot, *n the
// number of peaks (device memory, written between planner launches).
// n == nullptr: no batch.
constexpr int kMaxBatch = 32;       // aircraft of one co-simulated batch
constexpr int kMatePeaks = 5;       // peaks per aircraft
struct MatePeaks {
    const double *pk;
    const int *owner;
    const int *n;
};

// Device state of a co-simulated batch between planner launches.
struct BatchState {
    double *pk;
    int *owner, *n;
    int *active;     // aircraft flying in the step just planned
    int *prev_n;     // its point count before that step
    int *any;        // 1 while an aircraft is flying (pinned host memory)
};

// prop.mode selects the proposal path (FASTMDP_PROPOSE_NONE: full sweep
// only); the configuration, the launch's size and the outputs asked for select
// the kernel and its workgroup.
hipError_t launch_planner(int nblk, hipStream_t st, const DevCfg &c, const DevTable &t, Slot *s,
                          const int *list, const Traj &tr, int budget, int validate, int epoch, const EvalOut &ev,
                          const PropArgs &prop, const LaunchStop &stop, const MatePeaks &mates = MatePeaks{});

// batch.hip: after each planner step of a co-simulated batch (slots 0..n-1):
// separation between the aircraft that moved, goal capture and step limit,
// then the peaks of the aircraft still flying for the next step.  first:
// the launch before it only checked the origins.
hipError_t launch_batch_step(const DevCfg &c, Slot *slots, int n, const Traj &tr, const BatchState &bs, int first,
                             hipStream_t st);
bool planner_shape_supported(int n_climb, int n_speed, int zero_climb);

// Supported (climbs, speeds, zero-climb index) shapes of the planner kernels.
#define FMDP_PLANNER_SHAPES(X) \
    X(1, 1, 0) X(1, 1, -1) X(1, 2, 0) X(1, 2, -1) X(1, 3, 0) X(1, 3, -1) \
    X(2, 1, -1) X(2, 2, -1) X(2, 3, -1) \
    X(3, 1, 1) X(3, 1, -1) X(3, 2, 1) X(3, 2, -1) X(3, 3, 1) X(3, 3, -1) \
    X(5, 1, 2) X(5, 3, 2) X(5, 3, -1)

// range.hip: the range-query planner, kRangeThreads per request and
// kRangePerCU requests per compute unit, or kRangeThreadsSolo per request
// alone on a compute unit (full sweep with the range query, window W = 1,
// at most kRangeMaxHeads headings, no proposal, no co-simulated batch, no
// single-step outputs).
hipError_t launch_range_planner(int nblk, hipStream_t st, const DevCfg &c, const DevTable &t, Slot *s,
                                const int *list, const Traj &tr, int budget, int validate, int epoch,
                                const LaunchStop &stop);
// The full-sweep launches of this configuration go to the range-query
// planner.
inline bool uses_range_planner(const DevCfg &c, int prop_mode) {
    return c.range_query && c.lookahead <= 1 && prop_mode == FASTMDP_PROPOSE_NONE && c.n_head <= kRangeMaxHeads &&
           c.planner_threads != kPlanThreads;
}
// A launch of the full sweep of more requests than CUs takes two per CU
// (kPairThreads) unless the configuration asks for kPlanThreads, the longest
// row has more entries than that kernel holds at once, or the headings leave
// few slices a workgroup and the row is longer than a pair's tile.  Two
// requests that share a CU step 1.3 (1000 plans) to 1.6 times (3000) as
// slowly as alone, and past these limits up to 1.9 times, which a launch that
// waits for one long flight then takes: 400 departures, ms with pairs and
// without: 3000 plans, 81 actions 10.2 and 16.0; 5000 plans, 128 headings
// 55.7 and 41.9; 9000 plans, 360 actions 51.7 and 48.1.
inline bool uses_pairs(const DevCfg &c, int prop_mode) {
    return !c.range_query && c.lookahead <= 1 && prop_mode == FASTMDP_PROPOSE_NONE &&
           c.planner_threads != kPlanThreads && c.longest_row <= (c.n_head <= kPairHeads ? 2 : 1) * kPairTile;
}
// The range-query planner's workgroup size for a launch of nblk requests: as configured, else
// one request per CU on kRangeThreadsSolo threads when the launch holds no
// more requests than CUs, two to four per CU on kRangeThreads otherwise.
inline int range_planner_threads(const DevCfg &c, int nblk) {
    if (c.planner_threads == kRangeThreads || c.planner_threads == kRangeThreadsSolo) return c.planner_threads;
    return nblk <= c.n_cu ? kRangeThreadsSolo : kRangeThreads;
}

// features.hip: proposal features of n states (device arrays, see
// fastmdp_features).
// ws: features_workspace(rows) ints, or null (then one workgroup per state
// whatever n).  From kFeatGrouped states on they are grouped by row, a chunk
// at a time: a workgroup a state takes 5.7 us per 1000 states (51 us at 8000,
// 93 us at 16383), the groups and their order 82 us at 16384 (a workgroup for
// each CU; fewer states leave CUs idle at the same latency) and 114 us at
// 100000.
constexpr int kFeatChunk = 1 << 17, kFeatGrouped = 16384;
size_t features_workspace(int n_rows);
hipError_t launch_features(const DevCfg &c, const DevTable &t, int n, const double *states, const double *goals,
                           const int *rows, const int *seqs, float *feat, int *ws, hipStream_t st);

// mlp.hip: the planner's view of a network's weights.
int mlp_weights(const fastmdp_mlp *m, PropNet *w);

// table.hip
hipError_t launch_fill_int(int *p, int value, int n, hipStream_t st);
// The 16-bit coordinates of every place of the table (after points were read
// from a file).
hipError_t launch_quantise_table(const DevTable &t, hipStream_t st);
// Every row's grid over its longest prefix of entries that stay as they are:
// owned by sequence numbers below `limit` (accepted) or withdrawn.
hipError_t launch_build_grid(const DevTable &t, int limit, hipStream_t st);
hipError_t launch_scatter_points(const DevTable &t, const float *pts, const int *rows, const int *cols, int n,
                                 int own, hipStream_t st);
// Append n plans (t0[j], len[j], points plan-major in xyz; all device
// pointers) in order, each row's entries in plan order; the caller has
// checked rows and capacity.
hipError_t launch_append_plans(const DevTable &t, const int *t0, const int *len, int n, const float *xyz,
                               hipStream_t st);
// Commit of n points (host memory the device sees, or device memory): the
// check of each point into flags (n), then, if none refuses, the append;
// *result (the same kinds of memory): bit 0 conflict, bit 1 capacity.
hipError_t launch_commit(const DevCfg &c, const DevTable &t, const double *pts, int t0, int n, int seq, int *flags,
                         int *result, hipStream_t st);
// Pack listed slots' trajectories (points from off[i]) into dst: total*3
// doubles xyz, total doubles value, total ints action.  list, off and dst may
// be pinned host memory.
hipError_t launch_gather_traj(const Slot *slots, const int *list, int n_list, const long long *off, long long total,
                              const Traj &tr, void *dst, hipStream_t st);
// FCFS acceptance: launch_fcfs_begin once before a call's first planner
// launch (empty logs, row counts as they stand), then after each launch a
// pass over the admitted, not yet accepted slots in `list` (may be pinned host
// memory): tentative insert, interaction check, withdrawal (see table.hip).
// prev and cur are the logs of the pass before and of this one.
hipError_t launch_fcfs_begin(const DevTable &t, const PassBufs &pb, const DeathLog &a, const DeathLog &b,
                             hipStream_t st);
hipError_t launch_fcfs_pass(const DevCfg &c, const DevTable &t, Slot *slots, const int *list, int n_list,
                            const Traj &tr, const DeathLog &prev, const DeathLog &cur, const PassBufs &pb, int epoch,
                            hipStream_t st);
// Withdraw every table entry of the listed slots owned by sequence numbers
// from min_own on (an interrupted FCFS call).
hipError_t launch_fcfs_abort(const DevTable &t, Slot *slots, const int *list, int n_list, const Traj &tr, int min_own,
                             int epoch, hipStream_t st);

}  // namespace fmdp
