// Ranked downstream positions: a variant of the estimate in which a request does not join the
// back of every later queue but takes the place its budget gives it there.
//
// The paper keeps every worker queue in remaining-budget order (Section 3.3), so at a later
// stage i the requests ahead of a newcomer with deadline d are the ones that order serves first:
// those with deadline <= d under low budget first (the ones already there win ties), those with
// deadline >= d under high budget first, the whole queue in arrival order.  The estimate is
//   est = cost_k(pos) + max over the paths through k of sum over later stages i of cost_i(ahead_i(d))
// (Section 3.2 Eq.(4) and the DAG maximum), everything else as in the plain estimate.
//
// The kernels here run behind the ones that form the queues: those are sorted then, so ahead_i(d) is a
// binary search over queue i's slots (deadline looked up through order[]).  One thread per queue
// slot: neighbouring threads hold neighbouring deadlines of one queue, so their searches walk the
// same slots.  The downstream sum depends on the request now, so the path CSR is walked per
// request; the cost of each later stage is computed once per request and kept in LDS.
// Estimates of the plain call, where there are any, are overwritten: the on-chip kernel leaves them out for snapshots within
// the promise, and snapshots in queue order may be finished with their ranked estimates already (RankedArgs::todo).
#include "pard_device.hpp"

namespace pard {

namespace {

constexpr int kRThreads = 64;                          // one wave per workgroup: a thread's LDS row is private
constexpr unsigned long long kUnset = ~0ull;

// the queue g with seg_ptr[g] <= j < seg_ptr[g+1], among queues lo..hi
__device__ __forceinline__ int64_t queue_of(const int32_t* seg_ptr, int64_t lo, int64_t hi, int64_t j) {
    int64_t a = lo, b = hi + 1;                        // answer in [a, b)
    while (b - a > 1) {
        const int64_t mid = (a + b) >> 1;
        if ((int64_t)seg_ptr[mid] <= j) a = mid; else b = mid;
    }
    return a;
}

__global__ __launch_bounds__(kRThreads) void ranked_estimate_kernel(RankedArgs A) {
    extern __shared__ unsigned long long memo[];       // [S][kRThreads]: cost of later stage i for this thread's request
    const PlanDev& P = A.plan;
    const int tid = threadIdx.x;
    const int S = P.S;
    const int64_t segs = (int64_t)P.K * S;
    const int64_t tiles = (A.n + kRThreads - 1) / kRThreads;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t j0 = tile * kRThreads, j1 = j0 + kRThreads - 1 < A.n - 1 ? j0 + kRThreads - 1 : A.n - 1;
        const int64_t g_first = queue_of(A.seg_ptr, 0, segs - 1, j0), g_last = queue_of(A.seg_ptr, g_first, segs - 1, j1);
        const int64_t j = j0 + tid;
        if (j >= A.n) continue;
        const int64_t g = queue_of(A.seg_ptr, g_first, g_last, j);
        const int32_t u = (int32_t)(g / S), k = (int32_t)(g - (int64_t)u * S);
        const int64_t rec0 = P.shared ? 0 : (int64_t)u * S;
        const int32_t r = A.order[j];
        if ((uint32_t)r >= (uint64_t)A.n) continue;
        const int32_t d = A.deadline[r];
        for (int i = 0; i < S; ++i) memo[i * kRThreads + tid] = kUnset;
        const int32_t dag = P.shared ? 0 : u;
        const int32_t e_lo = P.dag_entry_ptr[dag], e_hi = P.dag_entry_ptr[dag + 1];
        unsigned long long best = 0;
        for (int32_t e = e_lo; e < e_hi; ++e) {
            if (P.entry_stage[e] != k) continue;
            const int32_t end = P.entry_end[e];
            unsigned long long sum = 0;
            for (int32_t t = e + 1; t < end; ++t) {
                const int32_t i = P.entry_stage[t];
                unsigned long long c = memo[i * kRThreads + tid];
                if (c == kUnset) {
                    const StageRec sr = P.recs[rec0 + i];
                    const int64_t start = A.seg_ptr[(int64_t)u * S + i], stop = A.seg_ptr[(int64_t)u * S + i + 1];
                    const int32_t mode = P.uniform_mode >= 0 ? P.uniform_mode : (sr.mode & 0xFF);
                    int64_t lo = start, hi = stop;     // first slot the newcomer does not have to let pass
                    if (mode == PARD_ORDER_FCFS) {
                        lo = stop;
                    } else {
                        while (lo < hi) {
                            const int64_t mid = (lo + hi) >> 1;
                            const int32_t rm = A.order[mid];
                            const int32_t dm = (uint32_t)rm < (uint64_t)A.n ? A.deadline[rm] : 0;
                            const bool passes = mode == PARD_ORDER_HBF ? dm >= d : dm <= d;
                            if (passes) lo = mid + 1; else hi = mid;
                        }
                    }
                    c = stage_cost(sr, (uint32_t)(lo - start), P.lat + (rec0 + i) * PARD_LAT_ENTRIES);
                    memo[i * kRThreads + tid] = c;
                }
                sum += c;
            }
            best = sum > best ? sum : best;
        }
        const StageRec own = P.recs[rec0 + k];
        const uint64_t e64 = stage_cost(own, (uint32_t)(j - (int64_t)A.seg_ptr[g]), P.lat + (rec0 + k) * PARD_LAT_ENTRIES) + best;
        int32_t est;
        uint8_t drp;
        finish_request(e64, A.now[u], d, est, drp);
        A.est[r] = est;
        A.drop[r] = drp;
    }
}

// Snapshots that fit LDS: one workgroup per snapshot first lays the deadlines out by queue slot
// in LDS, so a search step is one LDS read instead of two dependent global loads.
constexpr int kRSnapEntries = 1024;                    // path entries of a DAG kept in LDS (longer lists are read in place)

template <int kRSnapThreads>
__global__ __launch_bounds__(kRSnapThreads) void ranked_snapshot_kernel(RankedArgs A) {
    extern __shared__ unsigned long long lds[];         // memo [S][kRSnapThreads], then the deadlines by slot
    __shared__ StageRec recs[PARD_MAX_STAGES];
    __shared__ int32_t qstart[PARD_MAX_STAGES + 1];     // queue starts inside the snapshot
    __shared__ uint32_t ent[kRSnapEntries];             // stage | (end of the entry's path) << 8
    const PlanDev& P = A.plan;
    const int tid = threadIdx.x;
    const int S = P.S;
    unsigned long long* memo = lds;
    int32_t* dls = reinterpret_cast<int32_t*>(lds + (size_t)S * kRSnapThreads);
    const int32_t u = blockIdx.x;
    const int64_t a0 = A.seg_ptr[(int64_t)u * S], a1 = A.seg_ptr[(int64_t)(u + 1) * S];
    if (a0 < 0 || a1 < a0 || a1 > A.n || a1 - a0 > A.max_snapshot) return;   // larger than promised: reported by the plain call
    const int m = (int)(a1 - a0);
    const int64_t rec0 = P.shared ? 0 : (int64_t)u * S;
    const int32_t dag = P.shared ? 0 : u;
    const int32_t e_lo = P.dag_entry_ptr[dag], n_entries = P.dag_entry_ptr[dag + 1] - e_lo;
    const bool cached = n_entries <= kRSnapEntries;
    for (int j = tid; j < m; j += kRSnapThreads) {
        const int32_t r = A.order[a0 + j];
        dls[j] = (uint32_t)r < (uint64_t)A.n ? A.deadline[r] : 0;
    }
    {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(P.recs + rec0);
        uint32_t* dst = reinterpret_cast<uint32_t*>(recs);
        for (int i = tid; i < S * (int)(sizeof(StageRec) / 4); i += kRSnapThreads) dst[i] = src[i];
        for (int i = tid; i <= S; i += kRSnapThreads) qstart[i] = (int32_t)((int64_t)A.seg_ptr[(int64_t)u * S + i] - a0);
        if (cached)
            for (int e = tid; e < n_entries; e += kRSnapThreads)
                ent[e] = (uint32_t)P.entry_stage[e_lo + e] | ((uint32_t)(P.entry_end[e_lo + e] - e_lo) << 8);
    }
    __syncthreads();
    auto entry_stage = [&](int e) -> int { return cached ? (int)(ent[e] & 0xFFu) : P.entry_stage[e_lo + e]; };
    auto entry_end = [&](int e) -> int { return cached ? (int)(ent[e] >> 8) : P.entry_end[e_lo + e] - e_lo; };
    const int32_t now = A.now[u];
    for (int j = tid; j < m; j += kRSnapThreads) {
        int k = 0;                                      // the queue of slot j: the last one that starts at or before it
        while (k + 1 < S && qstart[k + 1] <= j) ++k;
        const int32_t d = dls[j];
        for (int i = 0; i < S; ++i) memo[i * kRSnapThreads + tid] = kUnset;
        unsigned long long best = 0;
        for (int e = 0; e < n_entries; ++e) {
            if (entry_stage(e) != k) continue;
            const int end = entry_end(e);
            unsigned long long sum = 0;
            for (int t = e + 1; t < end; ++t) {
                const int i = entry_stage(t);
                unsigned long long c = memo[i * kRSnapThreads + tid];
                if (c == kUnset) {
                    const int start = qstart[i], stop = qstart[i + 1];
                    const int32_t mode = P.uniform_mode >= 0 ? P.uniform_mode : (recs[i].mode & 0xFF);
                    int lo = start, hi = stop;           // first slot the newcomer does not have to let pass
                    if (mode == PARD_ORDER_FCFS) {
                        lo = stop;
                    } else {
                        while (lo < hi) {
                            const int mid = (lo + hi) >> 1;
                            const int32_t dm = dls[mid];
                            const bool passes = mode == PARD_ORDER_HBF ? dm >= d : dm <= d;
                            if (passes) lo = mid + 1; else hi = mid;
                        }
                    }
                    c = stage_cost(recs[i], (uint32_t)(lo - start), P.lat + (rec0 + i) * PARD_LAT_ENTRIES);
                    memo[i * kRSnapThreads + tid] = c;
                }
                sum += c;
            }
            best = sum > best ? sum : best;
        }
        const uint64_t e64 = stage_cost(recs[k], (uint32_t)(j - qstart[k]), P.lat + (rec0 + k) * PARD_LAT_ENTRIES) + best;
        const int32_t r = A.order[a0 + j];
        if ((uint32_t)r >= (uint64_t)A.n) continue;
        int32_t est;
        uint8_t drp;
        finish_request(e64, now, d, est, drp);
        A.est[r] = est;
        A.drop[r] = drp;
    }
}

// Pipelines of at most 16 stages whose snapshots fit LDS: a wave takes 64 slots of ONE queue, so everything about the
// pipeline is the same for its lanes: lane p of a wave holds the constants of the stage at place p, a read of one lane
// hands them to all.  The maximum over the paths is formed stage by stage (places rise away from the sinks) instead of
// path by path.  A search starts from a table per queue of where every 2^shift-th deadline value of the snapshot's range
// begins: one or two LDS steps are left of the binary search's eleven.  The table costs two bytes per bucket, a bucket
// holds about one slot of a queue.  Saturating 32-bit sums are enough: 2^32 - 1 and everything above it is past INT32_MAX
// as an estimate and past every deadline that can be exceeded, even from the lowest `now`.  Bound by vector instructions
// and dependent LDS reads (about 230 and 24 per 64 slots at 6 stages).  4096 snapshots of 8192, in order under low budget
// first: 354 us, 967 with a binary search over the whole queue and a walk of the paths per request (more than 16 stages still
// take that: ranked_snapshot_kernel).  Such snapshots are finished ahead of this kernel now (todo); in order under high budget
// first it takes 360 us, out of order 541 under either, where neighbouring slots hold requests from all over the snapshot.
__device__ __forceinline__ uint32_t sat32(uint64_t c) { return c < 0xFFFFFFFFull ? (uint32_t)c : 0xFFFFFFFFu; }
__device__ __forceinline__ int from_lane(int v, int l) { return __builtin_amdgcn_readlane(v, l); }

// FAST: every stage admits the 32-bit short-queue form of the cost (see stage_cost_short).
template <int NS, int T, bool FAST>
__global__ __launch_bounds__(T) void ranked_queues_kernel(RankedArgs A, int cap, int bucket_bits) {
    extern __shared__ int32_t dls[];                    // the deadlines by slot [cap], then the tables [S][buckets + 1]
    __shared__ StageRec recs[NS];
    __shared__ __align__(16) uint32_t quick[NS][8];     // by place: B-1, 1/B, 1/W, aW, bW, the queue's start, its length, the stage
    __shared__ int32_t lat[NS * PARD_LAT_ENTRIES];
    __shared__ int32_t edge[2][T / kWave];
    const PlanDev& P = A.plan;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = P.S, buckets = 1 << bucket_bits;
    uint16_t* table = reinterpret_cast<uint16_t*>(dls + cap);
    const int32_t u = blockIdx.x;
    const uint32_t marked = A.todo ? A.todo[u] : 1u;    // 0: came in queue order, its estimates are the ranked ones already
    const int64_t a0 = A.seg_ptr[(int64_t)u * S], a1 = A.seg_ptr[(int64_t)(u + 1) * S];
    if (a0 < 0 || a1 < a0 || a1 > A.n || a1 - a0 > A.max_snapshot) return;   // larger than promised: reported by the plain call
    if (a1 == a0 || marked == 0u) return;
    const int64_t rec0 = P.shared ? 0 : (int64_t)u * S;
    // lane i: where queue i starts (lane S: the end); lane p: the stage at place p, its queue's start and length, its order
    const int at = (int)((int64_t)A.seg_ptr[(int64_t)u * S + (lane < S ? lane : S)] - a0);
    const uint32_t topo = P.topo[(rec0 + (lane < S ? lane : 0)) * 2], later = P.topo[(rec0 + (lane < S ? lane : 0)) * 2 + 1];
    const int stage_p = (int)(topo & 0xFFu);
    const int mode_p = P.uniform_mode >= 0 ? P.uniform_mode : P.recs[rec0 + stage_p].mode & 0xFF;
    const int start_p = __shfl(at, stage_p), len_p = __shfl(at, stage_p + 1) - start_p;
    for (int i = tid; i < S * (int)(sizeof(StageRec) / 4); i += T)
        reinterpret_cast<uint32_t*>(recs)[i] = reinterpret_cast<const uint32_t*>(P.recs + rec0)[i];
    for (int i = tid; i < S * PARD_LAT_ENTRIES; i += T) lat[i] = P.lat[rec0 * PARD_LAT_ENTRIES + i];
    if (wave == 0 && lane < S) {
        const StageRec& r = P.recs[rec0 + stage_p];
        *reinterpret_cast<uint4*>(&quick[lane][0]) = make_uint4((uint32_t)r.B - 1u, __float_as_uint(r.rcpB), __float_as_uint(r.rcpW), r.aW);
        *reinterpret_cast<uint4*>(&quick[lane][4]) = make_uint4(r.bW, (uint32_t)start_p, (uint32_t)len_p, (uint32_t)stage_p);
    }
    const int32_t now = A.now[u];
    // the wave's share of the 64-slot chunks, queue by queue: a run of neighbouring ones
    int chunks = 0;
    for (int i = 0; i < S; ++i) chunks += (from_lane(at, i + 1) - from_lane(at, i) + 63) >> 6;
    const int c_lo = chunks * wave / (T / kWave), c_hi = chunks * (wave + 1) / (T / kWave);
    int k0 = 0, before0 = 0;                            // the first chunk's queue, and the chunks of the queues before it
    while (k0 < S) {
        const int here = (from_lane(at, k0 + 1) - from_lane(at, k0) + 63) >> 6;
        if (c_lo - before0 < here) break;
        before0 += here;
        ++k0;
    }
    // cost of the stage at a place with `ahead` requests ahead (below 2^13)
    auto cost_at = [&](const uint4& a, const uint4& b, uint32_t ahead) -> uint32_t {
        if (FAST) {
            const uint32_t q = (uint32_t)(((float)(ahead + a.x) + 0.5f) * __uint_as_float(a.y));
            const uint32_t wait = __umul24(q, a.w) + (uint32_t)(((float)__umul24(q, b.x) + 0.5f) * __uint_as_float(a.z));
            return wait + (uint32_t)lat[b.w * PARD_LAT_ENTRIES + (ahead < a.x ? ahead : a.x)];
        }
        return sat32(stage_cost_short(recs[b.w], ahead, lat + b.w * PARD_LAT_ENTRIES));
    };
    // every chunk of the share: f(queue, its start, its length, slot of this lane inside the queue)
    auto each_chunk = [&](auto f) {
        int k = k0, before = before0;
        for (int c = c_lo; c < c_hi; ++c) {
            int begin = from_lane(at, k), len = from_lane(at, k + 1) - begin;
            while (c - before >= (len + 63) >> 6) {     // c < chunks: there is such a queue
                before += (len + 63) >> 6;
                ++k;
                begin = from_lane(at, k);
                len = from_lane(at, k + 1) - begin;
            }
            f(k, begin, len, (c - before) * kWave + lane);
        }
    };
    int32_t low = kInt32Max, high = -kInt32Max - 1;
    {
        constexpr int U = 4;
        const int m = (int)(a1 - a0);
        for (int j0 = tid; j0 < m; j0 += U * T) {
            int32_t r[U], d[U];
#pragma unroll
            for (int x = 0; x < U; ++x) r[x] = A.order[a0 + (j0 + x * T < m ? j0 + x * T : j0)];
#pragma unroll
            for (int x = 0; x < U; ++x) d[x] = (uint32_t)r[x] < (uint64_t)A.n ? A.deadline[r[x]] : 0;
#pragma unroll
            for (int x = 0; x < U; ++x) {
                if (j0 + x * T < m) dls[j0 + x * T] = d[x];
                low = d[x] < low ? d[x] : low;
                high = d[x] > high ? d[x] : high;
            }
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const int32_t l2 = __shfl_xor(low, off), h2 = __shfl_xor(high, off);
        low = l2 < low ? l2 : low;
        high = h2 > high ? h2 : high;
    }
    if (lane == 0) { edge[0][wave] = low; edge[1][wave] = high; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < T / kWave; ++w) {
        low = edge[0][w] < low ? edge[0][w] : low;
        high = edge[1][w] > high ? edge[1][w] : high;
    }
    low = __builtin_amdgcn_readfirstlane(low);
    high = __builtin_amdgcn_readfirstlane(high);
    const uint32_t range = (uint32_t)high - (uint32_t)low;
    const int range_bits = range ? 32 - __clz((int)range) : 0;
    const int shift = range_bits > bucket_bits ? range_bits - bucket_bits : 0;
    auto bucket = [&](int mode, int32_t d) { return (mode == PARD_ORDER_HBF ? (uint32_t)high - (uint32_t)d : (uint32_t)d - (uint32_t)low) >> shift; };
    // where every bucket begins: the slot before and the slot itself say which buckets begin at it, and those behind the
    // last slot's begin at the queue's end.  A run of 64 or more (a far deadline leaves most buckets empty) is written by
    // the whole wave; shorter ones cost less side by side (from 6 on by the wave: one snapshot of 6051 in bursts 66 -> 75 us).
    each_chunk([&](int k, int begin, int len, int pos) {
        const int mode = P.uniform_mode >= 0 ? P.uniform_mode : __builtin_amdgcn_readfirstlane(recs[k].mode) & 0xFF;
        if (mode == PARD_ORDER_FCFS) return;
        uint16_t* row = table + k * (buckets + 1);
        const int last = pos < len ? (int)bucket(mode, dls[begin + pos]) : pos == len ? buckets : -1;
        int first = __builtin_amdgcn_update_dpp(0, last, 0x138, 0xF, 0xF, false) + 1;       // wave_shr:1, the slot before
        if (lane == 0) first = pos > 0 ? (int)bucket(mode, dls[begin + pos - 1]) + 1 : 0;
        auto fill = [&](int from, int to, int slot) { for (int b = from + lane; b <= to; b += kWave) row[b] = (uint16_t)slot; };
        constexpr int kRun = kWave;
        unsigned long long runs = __ballot(last - first >= kRun);
        if (last - first < kRun) for (int b = first; b <= last; ++b) row[b] = (uint16_t)pos;
        while (runs) {
            const int l = __builtin_ctzll(runs);
            runs &= runs - 1ull;
            fill(from_lane(first, l), from_lane(last, l), from_lane(pos, l));
        }
        if (from_lane(pos, kWave - 1) == len - 1) fill(from_lane(last, kWave - 1) + 1, buckets, len);
    });
    __syncthreads();
    each_chunk([&](int k, int begin, int len, int pos) {
        asm volatile("" ::: "memory");                  // the stages' constants are read again for every chunk: kept, they cost 64 registers
        const bool live = pos < len;
        const int j = begin + (live ? pos : 0);
        const int32_t r = A.order[a0 + j];
        const int32_t d = dls[j];
        const int own = (from_lane((int)topo, k) >> 8) & 0xFF;
        const uint32_t wanted = (uint32_t)from_lane((int)later, own);
        uint32_t behind[NS];                            // from a stage on to the end, on its longest way
#pragma unroll
        for (int p = 0; p < NS; ++p) {
            behind[p] = 0u;
            if (!((wanted >> p) & 1u)) continue;
            const uint32_t word = (uint32_t)from_lane((int)topo, p);
            const uint4 qa = *reinterpret_cast<const uint4*>(&quick[p][0]), qb = *reinterpret_cast<const uint4*>(&quick[p][4]);
            const int mode = from_lane(mode_p, p);
            uint32_t lo = qb.z;                         // first slot the newcomer does not have to let pass
            if (mode != PARD_ORDER_FCFS && from_lane(len_p, p) > 0) {
                const int32_t flip = mode == PARD_ORDER_HBF ? -1 : 0;
                const uint16_t* row = table + (int)(word & 0xFFu) * (buckets + 1) + bucket(mode, d);
                lo = row[0];
                uint32_t hi = row[1];
                const int32_t key = d ^ flip;
                const int32_t* queue = dls + qb.y;
                while (lo < hi) {
                    const uint32_t mid = (lo + hi) >> 1;
                    const bool passes = (queue[mid] ^ flip) <= key;
                    lo = passes ? mid + 1u : lo;
                    hi = passes ? hi : mid;
                }
            }
            uint32_t best = 0;
#pragma unroll
            for (int q = 0; q < p; ++q)
                if ((word >> (16 + q)) & 1u) best = behind[q] > best ? behind[q] : best;
            behind[p] = __builtin_elementwise_add_sat(cost_at(qa, qb, lo), best);
        }
        uint32_t best = 0;
        const uint32_t next = (uint32_t)from_lane((int)topo, own) >> 16;
#pragma unroll
        for (int q = 0; q < NS; ++q)
            if ((next >> q) & 1u) best = behind[q] > best ? behind[q] : best;
        const uint4 qa = *reinterpret_cast<const uint4*>(&quick[own][0]), qb = *reinterpret_cast<const uint4*>(&quick[own][4]);
        const uint32_t e32 = __builtin_elementwise_add_sat(cost_at(qa, qb, (uint32_t)(j - begin)), best);
        if (!live || (uint32_t)r >= (uint64_t)A.n) return;
        int32_t est;
        uint8_t drp;
        finish_request(e32, now, d, est, drp);
        A.est[r] = est;
        A.drop[r] = drp;
    });
}

}  // namespace

hipError_t launch_ranked(const RankedArgs& a, hipStream_t stream) {
    if (a.plan.S == 1) return hipSuccess;              // no later queue: the plain call's estimates are the ranked ones
    if (a.n <= 0) return hipSuccess;
    // the largest workgroup whose per-thread rows and the snapshot's deadlines fit 64 KB of LDS
    const int64_t cap = a.max_snapshot < 1 ? 1 : a.max_snapshot;
    auto lds_bytes = [&](int threads) { return (size_t)a.plan.S * threads * sizeof(unsigned long long) + (size_t)((cap + 1) & ~(int64_t)1) * 4; };
    if (a.max_snapshot <= PARD_FUSED_SNAPSHOT_CAPACITY && a.plan.S <= kTopoStages) {
        // About one slot of a queue to a bucket, at most 1024 (512 from 9 stages on: the tables then take 16 KB).  Threads
        // as for the general on-chip kernel: 16 slots each, fewer for the smallest snapshots.  Eight stages or 16, with and
        // without the short cost form: unrolled for more places than there are stages the kernel needs more registers and
        // skips the rest one by one (1000 snapshots of 4000, three stages with 300 workers: 99 us with 16 places, 87 with 8;
        // a search of the whole queue and a walk of the paths 96).  Where it gains least that search is still as fast or a
        // little faster: two stages with 300 workers, 5000 snapshots of 700 89 and 88 us, 30,000 of 200 155 and 151; 5000 of
        // 700 in two queues with one deadline far from all others 376 and 366.
        const bool few = a.plan.S <= 8;
        int bits = 4;
        while (bits < (few ? 10 : 9) && ((int64_t)8 << bits) < cap) ++bits;
        const int slots = (int)((cap + 3) & ~(int64_t)3);
        const size_t lds = (size_t)slots * 4 + (size_t)a.plan.S * ((1 << bits) + 1) * 2;
        const unsigned K = (unsigned)a.plan.K;
        auto launch = [&](auto kernel, int threads) { kernel<<<K, threads, lds, stream>>>(a, slots, bits); };
        if (few && a.plan.presorted_ok) {
            if (cap > 2048) launch(ranked_queues_kernel<8, 512, true>, 512);
            else if (cap > 512) launch(ranked_queues_kernel<8, 256, true>, 256);
            else launch(ranked_queues_kernel<8, 128, true>, 128);
        } else if (few) {
            if (cap > 2048) launch(ranked_queues_kernel<8, 512, false>, 512);
            else if (cap > 512) launch(ranked_queues_kernel<8, 256, false>, 256);
            else launch(ranked_queues_kernel<8, 128, false>, 128);
        } else if (a.plan.presorted_ok) {
            if (cap > 2048) launch(ranked_queues_kernel<kTopoStages, 512, true>, 512);
            else if (cap > 512) launch(ranked_queues_kernel<kTopoStages, 256, true>, 256);
            else launch(ranked_queues_kernel<kTopoStages, 128, true>, 128);
        } else {
            if (cap > 2048) launch(ranked_queues_kernel<kTopoStages, 512, false>, 512);
            else if (cap > 512) launch(ranked_queues_kernel<kTopoStages, 256, false>, 256);
            else launch(ranked_queues_kernel<kTopoStages, 128, false>, 128);
        }
        return hipGetLastError();
    }
    if (a.max_snapshot <= PARD_FUSED_SNAPSHOT_CAPACITY) {
        const unsigned K = (unsigned)a.plan.K;
        if (lds_bytes(512) <= 64 * 1024 && cap > 2048) { ranked_snapshot_kernel<512><<<K, 512, lds_bytes(512), stream>>>(a); return hipGetLastError(); }
        if (lds_bytes(256) <= 64 * 1024 && cap > 512) { ranked_snapshot_kernel<256><<<K, 256, lds_bytes(256), stream>>>(a); return hipGetLastError(); }
        if (lds_bytes(128) <= 64 * 1024) { ranked_snapshot_kernel<128><<<K, 128, lds_bytes(128), stream>>>(a); return hipGetLastError(); }
    }                                                   // else: many stages, the general kernel
    int64_t grid = (a.n + kRThreads - 1) / kRThreads;
    if (grid > 64 * (int64_t)a.num_cus) grid = 64 * (int64_t)a.num_cus;
    ranked_estimate_kernel<<<(unsigned)grid, kRThreads, (size_t)a.plan.S * kRThreads * sizeof(unsigned long long), stream>>>(a);
    return hipGetLastError();
}

}  // namespace pard
