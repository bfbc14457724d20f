// Device-side view of a plan and the small arithmetic helpers every kernel shares.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pard_host.hpp"

namespace pard {

constexpr int kWave = 64;
constexpr uint64_t kCostCap = (uint64_t)1 << 40;   // per-term clamp, see stage_cost()
constexpr int32_t kInt32Max = 0x7fffffff;

// Plan tables in device memory (passed to kernels by value).
struct PlanDev {
    int32_t K, S, shared, any_fcfs;
    int32_t uniform_mode;              // >= 0 when all stages share one order mode
    int32_t max_entries_per_dag;
    int32_t presorted_ok;              // every stage admits the 32-bit short-queue form (see HostPlan)
    const StageRec* recs;              // [D*S]
    const int32_t* lat;                // [D*S*64]
    const int32_t* dag_entry_ptr;      // [D+1]
    const int32_t* entry_stage;        // [E]
    const int32_t* entry_end;          // [E]
    const int32_t* entry_dag;          // [E]
    const uint32_t* topo;              // [D*S*2] order of the stages for a maximum over paths, S <= kTopoStages (see HostPlan)
    const int64_t* split_in;           // [D*S] per-module SLO split: longest way in (see HostPlan)
    const int64_t* split_whole;        // [D*S] longest whole path through the stage
    int64_t total_entries;             // E
};

// Status bits a kernel may raise in the workspace's status word.
enum : uint32_t {
    kStatusSnapshotTooLarge = 1u       // a snapshot exceeded the promised bound
};

__device__ __forceinline__ uint32_t magic_div_dev(uint32_t n, uint32_t m, uint32_t sh) {
    uint32_t t = __umulhi(m, n);
    return (t + ((n - t) >> (sh & 0xFF))) >> (sh >> 8);
}

// int32 -> uint32 preserving order, then the per-mode queue key: ascending key order
// is the queue order (Section 3.3: LBF = smallest remaining budget first, HBF = largest).
__device__ __forceinline__ uint32_t order_key(int32_t mode, int32_t deadline, int32_t arrival) {
    uint32_t d = (uint32_t)deadline ^ 0x80000000u;
    if (mode == PARD_ORDER_HBF) return ~d;
    if (mode == PARD_ORDER_FCFS) return (uint32_t)arrival ^ 0x80000000u;
    return d;
}

__device__ __forceinline__ int32_t clamp_stage(int32_t s, int32_t S) {
    return s < 0 ? 0 : (s >= S ? S - 1 : s);
}

// 64-bit by 32-bit division, kept out of line: it is long and almost never taken.
static __device__ __noinline__ uint64_t wide_div(uint64_t x, uint32_t d) { return x / d; }

// Eq.(2) in snapshot form with `a` requests ahead (0 <= a < 2^31):
//   floor(ceil(a/B) * lat[B] / W) + lat[min(B, a+1)]
// clamped to 2^40.  With lat[B] = aW * W + bW (bW < W) and q batches ahead, floor(q * lat[B] / W) is
// q * aW + floor(q * bW / W): what is left to divide fits 32 bits unless W is huge, while q * lat[B] itself
// passes 2^32 as soon as a queue is long.  Clamping every term at 2^40 keeps 64-bit sums of up to 65 terms
// exact-or-saturated: any sum that reaches the clamp is far above INT32_MAX even after
// adding the most negative `now`, so the reported estimate and the drop decision are
// the same as with unbounded integers.
__device__ __forceinline__ uint64_t stage_cost(const StageRec& r, uint32_t a, const int32_t* lat_row) {
    uint32_t q = magic_div_dev(a + (uint32_t)r.B - 1u, r.mB, r.shB);
    const uint64_t p = (uint64_t)q * r.bW;
    uint64_t wait = (uint64_t)q * r.aW;
    if ((p >> 32) == 0) wait += magic_div_dev((uint32_t)p, r.mW, r.shW);
    else wait += wide_div(p, (uint32_t)r.W);
    uint32_t ex = (a + 1u >= (uint32_t)r.B) ? (uint32_t)r.latB : (uint32_t)lat_row[a];
    uint64_t c = wait + ex;
    return c < kCostCap ? c : kCostCap;
}

// The same cost for a short queue (a < 2^13), without 32x32 multiplies or integer
// division when the stage allows it (kStageFast):
//   q = ceil(a/B) = trunc((a + B - 1 + 0.5) * (1/B))        exact: the true value sits at
//       least 0.5/B from an integer and the two float roundings move it by < 0.002 * 0.5/B
//   latB = aW*W + bW  =>  floor(q*latB/W) = q*aW + floor(q*bW/W)
//   p = q*bW < 2^21 (bW < W <= 256), floor(p/W) = trunc((p + 0.5) * (1/W))   exact: p + 0.5
//       is a float, the true value sits at least 0.5/W from an integer, error < 0.25/W
//   q*aW < 2^31 (aW < 2^18), so everything fits 32 bits.
__device__ __forceinline__ uint64_t stage_cost_short(const StageRec& r, uint32_t a, const int32_t* lat_row) {
    if (r.mode & kStageFast) {
        const uint32_t q = (uint32_t)(((float)(a + (uint32_t)r.B - 1u) + 0.5f) * r.rcpB);
        const uint32_t p = __umul24(q, r.bW);
        const uint32_t wait = __umul24(q, r.aW) + (uint32_t)(((float)p + 0.5f) * r.rcpW);
        const uint32_t ex = (a + 1u >= (uint32_t)r.B) ? (uint32_t)r.latB : (uint32_t)lat_row[a];
        return (uint64_t)wait + ex;
    }
    return stage_cost(r, a, lat_row);
}

// est (clamped) and the drop decision from the 64-bit estimate:
//   drop = min(now + e64, INT32_MAX) > deadline.
// A deadline of INT32_MAX can never be exceeded by the clamped finish time; for any smaller
// deadline the clamp does not change the comparison.
__device__ __forceinline__ void finish_request(uint64_t e64, int32_t now, int32_t deadline,
                                               int32_t& est, uint8_t& drop) {
    est = e64 > (uint64_t)kInt32Max ? kInt32Max : (int32_t)e64;
    const int64_t fin = (int64_t)now + (int64_t)e64;
    drop = ((deadline != kInt32Max) & (fin > (int64_t)deadline)) ? 1 : 0;
}

__device__ __forceinline__ uint32_t lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Inclusive prefix sum across the 64 lanes of a wave, on the vector ALU's data-parallel
// primitives: four shifts inside each row of 16 lanes, then the last lane of rows 0 and 2 is
// added to rows 1 and 3, and lane 31 to the upper half.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);    // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);    // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);    // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);    // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);    // row_bcast:15 into rows 1, 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);    // row_bcast:31 into rows 2, 3
    return v;
}

// Minimum over the lanes below (INT32_MAX in lane 0), on the vector ALU's data-parallel primitives.
__device__ __forceinline__ int32_t wave_exclusive_min(int32_t v) {
    const int32_t inf = kInt32Max;
    int32_t x = __builtin_amdgcn_update_dpp(inf, v, 0x138, 0xF, 0xF, false);          // wave_shr:1: the lane below's value
    auto lower = [](int32_t a, int32_t b) { return a < b ? a : b; };
    x = lower(x, __builtin_amdgcn_update_dpp(inf, x, 0x111, 0xF, 0xF, false));         // row_shr:1
    x = lower(x, __builtin_amdgcn_update_dpp(inf, x, 0x112, 0xF, 0xF, false));         // row_shr:2
    x = lower(x, __builtin_amdgcn_update_dpp(inf, x, 0x114, 0xF, 0xF, false));         // row_shr:4
    x = lower(x, __builtin_amdgcn_update_dpp(inf, x, 0x118, 0xF, 0xF, false));         // row_shr:8
    x = lower(x, __builtin_amdgcn_update_dpp(inf, x, 0x142, 0xA, 0xF, false));         // row_bcast:15 into rows 1, 3
    x = lower(x, __builtin_amdgcn_update_dpp(inf, x, 0x143, 0xC, 0xF, false));         // row_bcast:31 into rows 2, 3
    return x;
}

// How many positions, from 0 on, a request is in time at: positions with cost <= budget, for a stage whose cost never
// falls with the position and admits the short-queue form (pos < 2^13).  quick: the stage's row, lat: its latency table.
// Behind the first batch the cost is floor(q lat[B] / W) + lat[B] with q = ceil(pos / B), so q < (budget - lat[B] + 1) W / lat[B]:
// a float quotient, off by less than 0.01, and one exact comparison to either side.  In the first batch the wait is that
// of one batch and the execution one of B table entries.
// positions_from: the same for a budget b of at least lat[0].
__device__ __forceinline__ uint32_t positions_from(const uint32_t* quick, float inv, const uint32_t* lat, uint32_t b) {
    const uint4 qa = *reinterpret_cast<const uint4*>(quick);
    const uint32_t bW = quick[4];
    auto wait = [&](uint32_t q) { return __umul24(q, qa.w) + (uint32_t)(((float)__umul24(q, bW) + 0.5f) * __uint_as_float(qa.z)); };
    const uint32_t full = lat[qa.x], first = wait(1u);
    if (b < full || b - full < first) {                // not in time behind the whole first batch
        if (b < first) return 1u;
        uint32_t lo = 1u, hi = qa.x + 1u;              // table entries 1 .. B-1: the first that is too long
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (lat[mid] <= b - first) lo = mid + 1u; else hi = mid;
        }
        return lo;
    }
    const uint32_t room = b - full;                    // the longest wait that is in time
    uint32_t q = (uint32_t)fminf(((float)room + 1.0f) * inv, 8190.0f);
    if (wait(q) > room) --q;
    else if (wait(q + 1u) <= room) ++q;
    return q * (qa.x + 1u) + 1u;
}

__device__ __forceinline__ uint32_t positions_in_time(const uint32_t* quick, float inv, const uint32_t* lat, int64_t budget) {
    if (budget < (int64_t)lat[0]) return 0u;
    return positions_from(quick, inv, lat, budget < 0xFFFFFFFFll ? (uint32_t)budget : 0xFFFFFFFFu);         // every cost is below 2^32
}

// One step of a queue's chain under low budget first: 64 requests in queue order (`ok` in the lanes that hold one), c = how
// many positions a request is in time at, counted from the kept requests ahead of the 64.  Budgets rise along the queue, so
// does c, and the recurrence a' = min(a + 1, c) unrolls to a_i = min(i, i - 1 + min over i' < i of (c_i' - i')).  Returns the
// position and the mask of kept requests.
__device__ __forceinline__ int chain_step(bool ok, int c, int lane, unsigned long long& keep) {
    const int32_t least = wave_exclusive_min(c - lane);        // INT32_MAX for lane 0
    const int a = lane > 0 && least <= 0 ? lane - 1 + least : lane;
    keep = __ballot(ok && a < c);
    return a;
}

// Estimates and decisions are written once and not read again by the call that writes them: streaming stores
// (they leave the caches early and do not push out what the next kernel reads).
typedef int pard_v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void stream_store(int4* p, int4 v) {
    pard_v4i x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, reinterpret_cast<pard_v4i*>(p));
}
__device__ __forceinline__ void stream_store(uint32_t* p, uint32_t v) { __builtin_nontemporal_store(v, p); }

// Where a snapshot's staged survivors start inside the snapshot's own stretch of the staging array.  Snapshots
// of equal size start at equal distances; if every one staged its few survivors at its very start, they would
// all fall into the same few memory channels (measured: the kernel that moves them ran at an eighth of the
// bandwidth).  Eight consecutive snapshots therefore start at eight different eighths of the free room.
__host__ __device__ __forceinline__ uint32_t staging_shift(int64_t u, uint32_t requests, uint32_t survivors) {
    return ((uint32_t)(u & 7) * ((requests - survivors) >> 3)) & ~15u;
}

// ---- launchers implemented in the .hip files (host functions) ----------------

struct FusedArgs {
    PlanDev plan;
    const int32_t *arrival, *deadline, *stage, *snap_ptr, *now;
    int32_t *est;
    uint8_t* drop;
    int32_t *order, *seg_ptr;
    const int64_t* sub;                // [K*S] downstream latency per (snapshot, stage), or null: walk the paths
    uint32_t* status;
    uint32_t* todo;                    // [K] scratch, or null: snapshots left to the general kernel by the one for
                                       // snapshots that come in queue order
    // survivor compaction in the same pass (all three null otherwise):
    uint32_t* kept;                    // [K] out: survivors of every snapshot
    int32_t* staged;                   // [n] out: a snapshot's survivors in queue order from its first request's place on
    int32_t* loc_ptr;                  // [K*S] out: survivors of the snapshot before each of its queues
    int32_t cap;                       // promised bound on a snapshot's size
    int32_t consistent;                // positions count only the kept requests ahead
    int32_t ranked;                    // launch_ranked follows: the general kernel forms only the queues, the one for queue order the
                                       // ranked estimates of what it finishes where ranked_in_queue_order says so
    int64_t n;                         // total requests (bounds every index derived from snap_ptr)
    int32_t num_cus;
};
hipError_t launch_fused(const FusedArgs& a, hipStream_t stream);
// Ranked calls: whether the kernel for queue order tries first and finishes what it takes (todo[] then says which snapshots
// launch_ranked still has to do; else it does all of them).
bool ranked_in_queue_order(const FusedArgs& a);
// Snapshots whose requests already come in queue order (launch_fused tries this first when it applies).
constexpr int kPresortedMaxStages = 6;
bool presorted_path_covers(const FusedArgs& a);
hipError_t launch_presorted(const FusedArgs& a, hipStream_t stream);
// Snapshots of at most 128 requests, one wave each (launch_fused hands these over itself).
bool wave_path_covers(const FusedArgs& a);
hipError_t launch_wave(const FusedArgs& a, hipStream_t stream);

struct SortArgs {
    PlanDev plan;
    int64_t n;
    int64_t max_snapshot;              // promised bound on a snapshot's size
    const int32_t *arrival, *deadline, *stage, *snap_ptr, *now;
    int32_t* est;
    uint8_t* drop;
    int32_t *order, *seg_ptr;
    const int64_t* sub;                // as in FusedArgs
    int32_t consistent;                // as in FusedArgs
    uint32_t* status;
    void* workspace;                   // sort_workspace_bytes(K, S, n) bytes, 256-byte aligned
    int32_t num_cus;
};
int64_t sort_workspace_bytes(int32_t K, int32_t S, int64_t n);
bool sort_supported(int32_t K, int32_t S, int64_t n, int64_t max_snapshot);
hipError_t launch_sort_path(const SortArgs& a, hipStream_t stream);

struct RankedArgs {
    PlanDev plan;
    int64_t n;
    const int32_t *deadline, *now;
    const int32_t *order, *seg_ptr;    // the plain call's queues
    int32_t* est;                      // rewritten
    uint8_t* drop;
    const uint32_t* todo;              // [K], or null: only the snapshots marked here are still plain
    int64_t max_snapshot;              // promised bound on a snapshot's size
    int32_t num_cus;
};
hipError_t launch_ranked(const RankedArgs& a, hipStream_t stream);

struct CompactArgs {
    int32_t num_segments;              // K*S
    int32_t stages;                    // S
    int64_t max_snapshot;              // promised bound on a snapshot's size
    int64_t n;
    const int32_t *order, *seg_ptr;
    const uint8_t* drop;
    int32_t *surv_idx, *surv_ptr;
    uint32_t* status;
    void* workspace;
    int32_t num_cus;
    // after an estimate call that counted and staged the survivors along the way (all three null otherwise):
    const uint32_t* kept;              // [K] survivors per snapshot
    const int32_t* staged;             // [n] a snapshot's survivors in queue order, from its first request's place on
    const int32_t* loc_ptr;            // [K*S] survivors of the snapshot before each of its queues
};
// True when pard_compact gives every snapshot to one workgroup for this promised bound (the form the
// estimate kernels can prepare).
bool compact_per_snapshot(int64_t max_snapshot);
int64_t compact_workspace_bytes(int64_t n, int64_t num_snapshots);
hipError_t launch_compact(const CompactArgs& a, hipStream_t stream);

// ---- State Planner side (pard_planner.hip) ------------------------------------------
constexpr int kMaxWaitSamples = 16384;             // samples of the arrival process one workgroup holds in LDS
constexpr int32_t kMaxWaitLatency = 1 << 25;       // durations above this are not sampled (sums of 64 must fit 32 bits)

hipError_t launch_queue_lengths(const PlanDev& plan, int64_t n, const int32_t* stage, const int32_t* snap_ptr,
                                int32_t* qlen, hipStream_t stream);
struct SubArgs {
    PlanDev plan;
    const int32_t* qlen;               // [K*S]
    const int32_t* qdelay;             // [K*S] monitored queueing delays, or null: derived from qlen
    int32_t variant;                   // PARD_SUB_*
    int64_t rank;                      // 1-based order statistic of the sampled totals (full variant)
    int32_t num_samples;
    const int32_t* samples;            // [num_samples]
    const uint32_t* picks;             // [num_samples * S]
    uint32_t* drawn;                   // [S][samples, padded by stage sets] scratch: the arrival each (sample, stage) pair draws
    int32_t num_cus;
    unsigned long long* sub;           // [K*S] out
};
hipError_t launch_sub_latency(const SubArgs& a, hipStream_t stream);
hipError_t launch_priority_modes(const PlanDev& plan, int32_t series_len, int32_t window, const int32_t* rate,
                                 const int32_t* prev_mode, int32_t* mode_out, hipStream_t stream);
hipError_t launch_queue_delay(int32_t K, int32_t S, int32_t len, uint32_t window, const int32_t* time, const int32_t* delay,
                              const int32_t* now, int32_t* q, hipStream_t stream);
hipError_t launch_set_modes(StageRec* recs, const int32_t* modes, int64_t count, hipStream_t stream);

// ---- reactive policies (pard_reactive.hip) --------------------------------------------
hipError_t launch_window_scan(const PlanDev& plan, int64_t n, const int32_t* deadline, const int32_t* order, const int32_t* seg_ptr,
                              const int32_t* now, uint8_t* drop, int32_t* first, hipStream_t stream);
hipError_t launch_slo_split(const PlanDev& plan, int64_t n, const int32_t* arrival, const int32_t* deadline, const int32_t* stage,
                            const int32_t* snap_ptr, const int32_t* now, uint8_t* drop, hipStream_t stream);

}  // namespace pard
