// features.hip -- proposal features of a batch of states (training data and
// checks of the planner's in-loop features, which use the same helpers).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "planner.h"
#include "proposal.h"
#include "score.h"
#include "wave.h"

namespace fmdp {

namespace {

constexpr int kFeatThreads = 256;
constexpr int kFeatGroup = 64;           // states of one workgroup of the grouped kernel
constexpr int kFeatHits = 512;           // its list of (state, entry) pairs inside a box
static_assert(kFeatGroup == 64, "a wave holds a group's states; a pair packs the state in six bits");

// Half-width of the box test on x or y around the FP32 coordinate `at`: the
// features' radius plus the roundings of both FP32 coordinates.
__device__ __forceinline__ float feat_reach(float at) { return kFeatR + 1.0f + 4e-7f * fabsf(at); }

// Entry idx, if request `seq` sees it, into the accumulators of the state s
// with direction (ux, uy) to its goal: the offset q = p - s rounded to FP32
// exactly as the planner stages it.
__device__ __forceinline__ void feat_entry(FeatAcc &fa, const DevTable &tb, size_t idx, int seq, const double s[3],
                                           float ux, float uy) {
    if (!entry_visible(tb, idx, seq)) return;
    const float qx = (float)((double)tb.X[idx] - s[0]);
    const float qy = (float)((double)tb.Y[idx] - s[1]);
    const float qz = (float)((double)tb.Z[idx] - s[2]);
    feat_point(fa, qx, qy, qz >= 0.0f, fmaf(qx, qx, fmaf(qy, qy, qz * qz)), ux, uy);
}

__device__ __forceinline__ void feat_direction(const double s[3], const double g[3], float &ux, float &uy) {
    const double bx = g[0] - s[0], by = g[1] - s[1];
    const double r = sqrt(dot2(bx, bx, by, by));
    ux = (float)(r > 0.0 ? bx / r : 1.0);
    uy = (float)(r > 0.0 ? by / r : 0.0);
}

// Four consecutive entries' x and y from entry j of the row at rb; entries at
// or past n lie far off.  (A row's capacity is a multiple of four, so the
// group is in bounds whenever its first entry is.)
__device__ __forceinline__ void feat_load4(const DevTable &tb, size_t rb, int j, int n, float x[4], float y[4]) {
    float4 x4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), y4 = x4;
    if (j < n) {
        x4 = *reinterpret_cast<const float4 *>(tb.X + rb + j);
        y4 = *reinterpret_cast<const float4 *>(tb.Y + rb + j);
    }
    const float xs[4] = {x4.x, x4.y, x4.z, x4.w}, ys[4] = {y4.x, y4.y, y4.z, y4.w};
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        x[m] = j + m < n ? xs[m] : INFINITY;
        y[m] = ys[m];
    }
}

// One workgroup per state: the entries of row rows[i] + 1 visible to
// sequence number seqs[i].  Bound by latency at a few states: x and y are
// tested first, the other columns read for the few entries inside the box,
// and each wave computes its share of the goal and box features (one wave
// with all twelve, one branch behind the other, took longer than the row).
__global__ __launch_bounds__(kFeatThreads) void features_kernel(DevCfg c, DevTable tb, int n,
                                                                const double *__restrict__ states,
                                                                const double *__restrict__ goals,
                                                                const int *__restrict__ rows,
                                                                const int *__restrict__ seqs,
                                                                float *__restrict__ feat) {
    __shared__ FeatAcc fa;
    const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (i >= n) return;
    feat_reset(fa, tid);
    __syncthreads();
    const double s[3] = {states[3 * i], states[3 * i + 1], states[3 * i + 2]};
    const double g[3] = {goals[3 * i], goals[3 * i + 1], goals[3 * i + 2]};
    const int row = rows[i] + 1, seq = seqs[i];
    float ux, uy;
    feat_direction(s, g, ux, uy);
    const int n_row = (row >= 0 && row < tb.rows) ? min(tb.rowN[row], tb.cap) : 0;
    const size_t rb = (size_t)(row >= 0 ? row : 0) * tb.cap;
    const float sx = (float)s[0], sy = (float)s[1], rx = feat_reach(sx), ry = feat_reach(sy);
    for (int j = 4 * tid; j < n_row; j += 4 * kFeatThreads) {
        float x[4], y[4];
        feat_load4(tb, rb, j, n_row, x, y);
#pragma unroll
        for (int m = 0; m < 4; ++m)
            if (fabsf(x[m] - sx) < rx && fabsf(y[m] - sy) < ry) feat_entry(fa, tb, rb + j + m, seq, s, ux, uy);
    }
    __syncthreads();
    float *out = feat + (size_t)i * FASTMDP_N_FEAT;
    for (int f = 4 * kSectors + wave; f < kFeatUsed; f += kFeatThreads / 64) {      // uniform per wave
        const float v = feat_value(fa, f, s, g, c.box_lo, c.box_hi, c.ell);
        if (lane == 0) out[f] = v;
    }
    if (tid < 4 * kSectors) out[tid] = feat_value(fa, tid, s, g, c.box_lo, c.box_hi, c.ell);
    else if (tid < 4 * kSectors + FASTMDP_N_FEAT - kFeatUsed) out[tid - 4 * kSectors + kFeatUsed] = 0.0f;
}

// Grouping by row: each state's rank among the states of its row (the last
// bin: rows outside the table, which have no entries), the bins' offsets, and
// the states in bin order (any order within a bin: each state's features are
// its own).
__device__ __forceinline__ int feat_bin(int row, int n_rows) { return row >= 0 && row < n_rows ? row : n_rows; }

// The ranks' atomics on one row go one behind the other (11 ns each: 100000
// states of one row took 1.1 ms), so a wave takes one for all of its states
// of a row that many share, for the first such rows it holds; rows that few
// share are counted one by one.
__global__ void feat_rank_kernel(int n, const int *__restrict__ rows, int n_rows, int *count, int *rank) {
    constexpr int kShared = 8, kTries = 4;                // states of a row in the wave; rows tried
    const int i = blockIdx.x * blockDim.x + threadIdx.x, lane = threadIdx.x & 63;
    int bin = i < n ? feat_bin(rows[i] + 1, n_rows) : -1;
    uint64_t open = __ballot(bin >= 0);                   // states without a rank whose row was not tried
    for (int q = 0; q < kTries && open; ++q) {            // uniform
        const int lead = __builtin_ctzll(open), row = __shfl(bin, lead);
        const uint64_t same = __ballot(bin == row);
        open &= ~same;
        if (__popcll(same) < kShared) continue;
        int first = 0;
        if (lane == lead) first = atomicAdd(&count[row], __popcll(same));
        first = __shfl(first, lead);
        if (bin == row) {
            rank[i] = first + __popcll(same & ((1ull << lane) - 1));
            bin = -1;
        }
    }
    if (bin >= 0) rank[i] = atomicAdd(&count[bin], 1);
}

__global__ __launch_bounds__(1024) void feat_offset_kernel(int bins, const int *__restrict__ count, int *off) {
    __shared__ int part[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int carry = 0;
    for (int b0 = 0; b0 < bins; b0 += 1024) {             // uniform
        const int v = b0 + tid < bins ? count[b0 + tid] : 0;
        int sum = v;                                      // inclusive over the wave
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(sum, d);
            if (lane >= d) sum += o;
        }
        if (lane == 63) part[wave] = sum;
        __syncthreads();
        int before = carry, all = 0;
        for (int w = 0; w < 16; ++w) {
            before += w < wave ? part[w] : 0;
            all += part[w];
        }
        if (b0 + tid < bins) off[b0 + tid] = before + sum - v;
        carry += all;
        __syncthreads();
    }
}

__global__ void feat_order_kernel(int n, const int *__restrict__ rows, int n_rows, const int *__restrict__ off,
                                  const int *__restrict__ rank, int *order) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) order[off[feat_bin(rows[i] + 1, n_rows)] + rank[i]] = i;
}

// kFeatGroup states in row order per workgroup: a row's x and y are read once
// for the group's states of that row and tested against each in registers;
// the pairs inside a box (about four a state) are collected and scored
// together, one per lane, and the goal and box features are computed with a
// state per lane and a feature per wave.  Bound by the box tests (under four
// FP32 operations per state and entry) and, at few states a row, by the
// rows' latency; one workgroup a state read the row for itself and ended in
// one wave's twelve branches.  100000 states of 3000 plans: 688 us before,
// 87 us now and 26 us to group them (18 us of it the ranks' atomics).
__global__ __launch_bounds__(kFeatThreads) void features_group_kernel(DevCfg c, DevTable tb, int n,
                                                                      const int *__restrict__ order,
                                                                      const double *__restrict__ states,
                                                                      const double *__restrict__ goals,
                                                                      const int *__restrict__ rows,
                                                                      const int *__restrict__ seqs,
                                                                      float *__restrict__ feat) {
    constexpr int S = kFeatGroup;
    static_assert(4 * kSectors == 64, "one lane per sector feature");
    __shared__ FeatAcc fa[S];
    __shared__ float4 box[S];                             // x, y, half-width
    __shared__ double pos[S][3];
    __shared__ float2 dir[S];
    __shared__ int id[S], row_of[S], seq_of[S];
    __shared__ uint32_t hit[kFeatHits];                   // entry << 6 | state
    __shared__ int n_hit;
    __shared__ uint64_t s_heads;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i0 = blockIdx.x * S, ns = min(S, n - i0);
    for (int q = tid; q < S * 2 * kSectors; q += kFeatThreads) feat_reset(fa[q / (2 * kSectors)], q % (2 * kSectors));
    if (tid == 0) n_hit = 0;
    if (wave == 0) {
        const int i = order[i0 + min(lane, ns - 1)];
        const double s[3] = {states[3 * i], states[3 * i + 1], states[3 * i + 2]};
        const double g[3] = {goals[3 * i], goals[3 * i + 1], goals[3 * i + 2]};
        const int row = feat_bin(rows[i] + 1, tb.rows);
        float ux, uy;
        feat_direction(s, g, ux, uy);
        id[lane] = i;
        row_of[lane] = row;
        seq_of[lane] = seqs[i];
        for (int a = 0; a < 3; ++a) pos[lane][a] = s[a];
        dir[lane] = make_float2(ux, uy);
        const float sx = (float)s[0], sy = (float)s[1];
        box[lane] = make_float4(sx, sy, fmaxf(feat_reach(sx), feat_reach(sy)), 0.0f);
        const int before = __shfl_up(row, 1);
        const uint64_t heads = __ballot(lane < ns && (lane == 0 || before != row));
        if (lane == 0) s_heads = heads;
    }
    __syncthreads();
    const uint64_t heads = s_heads;
    auto score = [&](int k, int j) {
        feat_entry(fa[k], tb, (size_t)row_of[k] * tb.cap + j, seq_of[k], pos[k], dir[k].x, dir[k].y);
    };
    for (uint64_t h = heads; h; h &= h - 1) {             // uniform: the rows
        const int k0 = __builtin_ctzll(h), k1 = (h & (h - 1)) ? __builtin_ctzll(h & (h - 1)) : ns;
        const int row = row_of[k0];
        const int n_row = row < tb.rows ? min(tb.rowN[row], tb.cap) : 0;
        const size_t rb = (size_t)row * tb.cap;
        for (int j = 4 * tid; j < n_row; j += 4 * kFeatThreads) {
            float x[4], y[4];
            feat_load4(tb, rb, j, n_row, x, y);
            for (int k = k0; k < k1; ++k) {
                const float4 b = box[k];
                float d[4];
#pragma unroll
                for (int m = 0; m < 4; ++m) d[m] = fmaxf(fabsf(x[m] - b.x), fabsf(y[m] - b.y));
                if (!(fminf(fminf(d[0], d[1]), fminf(d[2], d[3])) < b.z)) continue;
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    if (d[m] < b.z) {
                        const int o = atomicAdd(&n_hit, 1);
                        if (o < kFeatHits) hit[o] = (uint32_t)(j + m) << 6 | (uint32_t)k;
                        else score(k, j + m);             // the list is full
                    }
            }
        }
    }
    __syncthreads();
    for (int o = tid; o < min(n_hit, kFeatHits); o += kFeatThreads) score(hit[o] & 63u, hit[o] >> 6);
    __syncthreads();
    const int i = id[lane];
    const double g[3] = {goals[3 * i], goals[3 * i + 1], goals[3 * i + 2]};
    for (int f = 4 * kSectors + wave; f < kFeatUsed; f += kFeatThreads / 64) {      // uniform per wave
        const float v = feat_value(fa[lane], f, pos[lane], g, c.box_lo, c.box_hi, c.ell);
        if (lane < ns) feat[(size_t)i * FASTMDP_N_FEAT + f] = v;
    }
    for (int k = wave; k < ns; k += kFeatThreads / 64) {  // 64 features and the padding, a state per wave
        float *out = feat + (size_t)id[k] * FASTMDP_N_FEAT;
        out[lane] = feat_value(fa[k], lane, pos[k], g, c.box_lo, c.box_hi, c.ell);
        if (lane < FASTMDP_N_FEAT - kFeatUsed) out[kFeatUsed + lane] = 0.0f;
    }
}

}  // namespace

size_t features_workspace(int n_rows) { return 2 * ((size_t)n_rows + 1) + 2 * (size_t)kFeatChunk; }

hipError_t launch_features(const DevCfg &c, const DevTable &t, int n, const double *states, const double *goals,
                           const int *rows, const int *seqs, float *feat, int *ws, hipStream_t st) {
    for (int i0 = 0; i0 < n; i0 += kFeatChunk) {
        const int m = std::min(n - i0, kFeatChunk);
        const double *ps = states + 3 * (size_t)i0, *pg = goals + 3 * (size_t)i0;
        const int *pr = rows + i0, *pq = seqs + i0;
        float *pf = feat + (size_t)i0 * FASTMDP_N_FEAT;
        if (!ws || m < kFeatGrouped || t.cap >= 1 << 26) {
            hipLaunchKernelGGL(features_kernel, dim3(m), dim3(kFeatThreads), 0, st, c, t, m, ps, pg, pr, pq, pf);
            continue;
        }
        const int bins = t.rows + 1;
        int *count = ws, *off = ws + bins, *rank = off + bins, *order = rank + kFeatChunk;
        const dim3 per((m + 255) / 256), blk(256);
        const hipError_t e = launch_fill_int(count, 0, bins, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(feat_rank_kernel, per, blk, 0, st, m, pr, t.rows, count, rank);
        hipLaunchKernelGGL(feat_offset_kernel, dim3(1), dim3(1024), 0, st, bins, count, off);
        hipLaunchKernelGGL(feat_order_kernel, per, blk, 0, st, m, pr, t.rows, off, rank, order);
        hipLaunchKernelGGL(features_group_kernel, dim3((m + kFeatGroup - 1) / kFeatGroup), dim3(kFeatThreads), 0, st,
                           c, t, m, order, ps, pg, pr, pq, pf);
    }
    return hipGetLastError();
}

}  // namespace fmdp
