// Internal declarations shared by the HIP translation units of libskrull_attn.
// Nothing here is part of the public ABI (that is include/skrull_attn.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "skrull_attn.h"

struct WorkQueue;
// forward calls of one plan that may be in flight at once (each takes one queue slot in turn)
#define SKRULL_FWD_QUEUE_SLOTS 64
#define SKRULL_QUEUE_INTS 256  // of a queue: eight dies' queues, a 128-byte line each
// of what the workgroups of a backward share: the queues of dQ and of dK/dV, counters, a line each, and one more for each
// (shared dK/dV item, KV head), up to a limit
#define SKRULL_ITEM_COUNTERS 1024
#define SKRULL_BWD_STATE_INTS (2 * SKRULL_QUEUE_INTS + 128 + SKRULL_ITEM_COUNTERS)

// Queues that need no kernel to clear them before a launch.  The calls of one stream run one after another, so a
// plan keeps two sets for its calls on the default stream: a launch works with one and clears the other, which the
// launch before it has left, for the next.  (With a kernel before each that clears its queue, forwards of 26,624 tokens in 64 sequences, 14/2 heads of 64, come 64.0 us
// apart, the last item of one and the first of the next 6.4; 63.0 and 4.7 without.)  Calls on other streams and calls that are
// being captured (a replay has no turn in that order) clear a queue first: a stream that a program has made it may destroy
// while its work is under way (hipStreamDestroy need not wait), and a later stream may have the same handle, so that calls with one handle
// are not always one after another.  The default stream cannot be destroyed.
#define SKRULL_SETS_INTS (2 * (SKRULL_QUEUE_INTS + SKRULL_BWD_STATE_INTS))
struct DefaultStream {
    std::mutex lock;            // held from the choice of a set until the launch that uses it is queued
    uint32_t fwd = 0, bwd = 0;  // forward and backward calls so far that used a set
    bool lost = false;          // a launch failed: nobody knows what its sets hold

    // Whether a call on `st` may use a set.  With the lock held.
    bool has(hipStream_t st) const
    {
        if (st != nullptr || lost) return false;
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &capture) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        return capture == hipStreamCaptureStatusNone;
    }
};

#define SKRULL_CHAIN_LIMITS 9
#define SKRULL_UNIT_SHIFT 11  // rank-sorted lists have at most 2,048 items
#define SKRULL_UNIT_LISTS 3   // of forward / dQ work: for workgroups of 4, 8 and (head_dim 64) 12 wavefronts
#define SKRULL_UNIT_HEADS 1024  // more query heads go without a list of units (index arithmetic of row_blocks)

// Device-resident descriptor + work lists of one micro-batch.
struct skrull_attn_plan {
    int32_t K, NS, Hq, Hkv, d, BM, BN;  // K sequences, NS >= K query segments
    float scale;
    int32_t total_q, total_k, n_fwd, n_dkv;
    int32_t longest_seq;  // tokens of the longest sequence, also where this rank has a slice of it
    int64_t pairs;
    int32_t head_split;  // workgroups that share the query heads of one KV group in dK/dV
    int32_t wg_query_rows;  // query rows per forward / dQ workgroup, asked for or chosen: 128 or 256; what runs follows
    int32_t fwd_waves, dq_waves;  // wavefronts of a forward / dQ workgroup: 4, 8 or 12
    bool dq_piped;                // dQ of 4: pipelined, two workgroups per compute unit
    bool dq_packed;               // in one launch with dK/dV of 12 wavefronts: dQ units of 12 row blocks whatever dq_waves is
    // dK/dV items that several workgroups share (the first n_split of the sorted list), and how:
    // an item of cost c takes min(split_parts, ceil(c * heads per group / split_chain)) of them
    // (split_chain 0: split_parts).  Where there is no list of units, n_whole_first more items are handed out before those.
    int32_t n_split, n_whole_first, split_parts, split_chain;
    int32_t split_compact;  // 1: partial sums hold the rows of split items only; 0: every row of K
    int device;
    // one allocation (descriptor arrays, then the two item lists); the pointers below index into it
    int32_t *pool;
    int32_t *cu_q, *cu_k, *q_begin, *q_len, *kv_len, *shares_kv;  // per segment: [NS+1] x2, [NS] x4
    int32_t *fwd_items, *dkv_items;                   // [n][4], sorted
    // work units of the forward / dQ list for workgroups of 4, 8 and 12 wavefronts (see RowMap): item |
    // part << SKRULL_UNIT_SHIFT, longest first (UnitCosts in plan.hip); null for lists too long
    // for the rank sort and for very many heads
    int32_t *units[SKRULL_UNIT_LISTS], n_units[SKRULL_UNIT_LISTS];
    // The same of the dK/dV list, or null: {segment, key block, item | part << SKRULL_UNIT_SHIFT, parts of the item}.
    // (With the item's position alone, each unit began with one more load that all its others waited for: dK/dV of 60
    // small launches takes 1.5 % more that way, of 40 micro-batches of long chains at head_dim 64 0.5 %.)
    int4 *dkv_units;
    int32_t n_dkv_units;
    WorkQueue *fwd_queues;  // SKRULL_FWD_QUEUE_SLOTS times eight dies' queues, at the start of the pool: for forward launches that clear one first
    int32_t *sets;          // SKRULL_SETS_INTS: two sets of a forward, two of a backward, zero when the plan is made (see DefaultStream)
    DefaultStream *default_stream;
    uint32_t fwd_calls;     // such calls made so far (atomic): call i uses slot i mod SKRULL_FWD_QUEUE_SLOTS
};

// Which dK/dV items several workgroups share, and how; see skrull_attn_plan.
struct SplitChoice {
    int32_t head_split, n_split, n_whole_first, parts, chain, compact;
};

// Totals written by the plan kernels and read back by the host.
struct PlanTotals {
    int64_t total_q, total_k, n_fwd, n_dkv, pairs;
    int32_t bad_entry;   // index+1 of the first invalid sequence, 0 if none
    int32_t n_seg;       // number of query segments
    // cost (query blocks) of the dK/dV items, accumulated by the emit kernel
    unsigned long long dkv_cost_sum;
    int32_t dkv_cost_max;
    // chains of dK/dV items (query blocks x heads of a group, walked one after another by a workgroup
    // that has the item to itself): how many exceed exactly the first k of dkv_chain_limit()
    int32_t chain_base, chain_hist[SKRULL_CHAIN_LIMITS + 1];
    int32_t n_units[SKRULL_UNIT_LISTS];  // work units of the forward / dQ list for 4, 8 and 12 wavefronts
    int32_t n_dkv_units;
    // forward work in workgroups of 12 wavefronts, in half tiles of keys: of all units of a KV head, of the longest one
    // (16 half tiles for a unit's start and end included), of the longest one of more than 128 rows of a head (0: none)
    int64_t fwd_load;
    int32_t fwd_longest, fwd_longest_full;
    SplitChoice split;         // how dK/dV items are shared (the units kernel's choice)
    int32_t cap_fwd, cap_dkv;  // room in the item arrays (the host's upper bounds)
    int32_t block_n;           // key rows per dK/dV item in effect (the ranges kernel's choice where open)
};

constexpr int32_t kMaxParts = 8;  // workgroups that may share one dK/dV item whose heads are not split

// Bytes of backward scratch without partial sums: -D and LSE*log2(e) per (head, row), then 256
// bytes for the work queues of the two kernels in calls that clear these first.
__host__ __device__ inline int64_t base_workspace(int32_t q_heads, int64_t total_q)
{
    return ((((int64_t)q_heads * total_q * 8) + 255) & ~(int64_t)255) + 256;
}

// fp32 partial dK and dV of the items that several workgroups share: a slot per part for every row of
// K, or for the rows of those items only.
__host__ __device__ inline int64_t partial_bytes(const SplitChoice &c, int32_t block_n, int64_t total_k, int32_t kv_heads, int32_t head_dim)
{
    if (c.parts <= 1) return 0;
    const int64_t rows = c.compact ? (int64_t)c.n_split * block_n : total_k;
    return 2 * (int64_t)c.parts * rows * kv_heads * head_dim * 4;
}

// The k-th of the limits that a dK/dV item's chain is compared with: `base` times 2^((k - 2) / 2).
__host__ __device__ inline int64_t dkv_chain_limit(int32_t base, int k)
{
    const int32_t c = (k & 1) ? 181 : 128;  // 256 / sqrt(2), 256 / 2
    return ((int64_t)base * c << (k >> 1)) >> 8;
}

// Opt-in per-workgroup trace (measurement aid): one record per work item of a launch.
struct WgTrace {
    uint64_t t0, t1;      // s_memrealtime (100 MHz, one counter for the whole chip) at start and end
    uint32_t hw_id;       // HW_ID register: bits 8-11 CU, 12 shader array, 13-15 shader engine
    uint32_t xcc_id;      // XCC_ID register: the die (XCD)
    uint32_t block;       // index of the work item (the block index in a plain grid)
    uint32_t one;         // 1 = record written
};
#ifdef __HIPCC__
__device__ __forceinline__ uint64_t trace_begin(const WgTrace *t)
{
    return t ? __builtin_amdgcn_s_memrealtime() : 0;
}
// every wave of the workgroup calls this at the very end of the kernel (wave-uniform branch)
__device__ __forceinline__ void trace_end(WgTrace *t, uint64_t t0, int work)
{
    if (!t) return;
    __syncthreads();
    if (threadIdx.x == 0) {
        WgTrace r;
        r.t0 = t0;
        r.t1 = __builtin_amdgcn_s_memrealtime();
        r.hw_id = __builtin_amdgcn_s_getreg((31 << 11) | 4);    // HW_REG_HW_ID, all 32 bits
        r.xcc_id = __builtin_amdgcn_s_getreg((31 << 11) | 20);  // HW_REG_XCC_ID
        r.block = work;
        // (formed here: as a constant it was kept, and spilled, through the whole work loop)
        asm volatile("v_mov_b32 %0, 1" : "=v"(r.one));
        t[work] = r;
    }
}
#endif

// plan.hip
// A plan made by one workgroup: at most SKRULL_SMALL_PLAN sequences, segments and items of either list (a thread each).
#define SKRULL_SMALL_PLAN 512
struct SmallPlan {
    const int32_t *in;      // pinned host memory: S, N, R, cut, `stride` ints apart
    PlanTotals *totals;     // pinned host memory
    int32_t K, stride, BM, BN, bn_alt, max_q_rows, max_k_rows, cap_fwd, cap_dkv;
    int32_t q_heads, kv_heads, head_dim, asked, longest_seq, compute_units;
    int32_t *q_begin, *q_len, *kv_len, *cu_q, *cu_k, *shares_kv, *fwd_items, *dkv_items;
    int32_t *units[SKRULL_UNIT_LISTS];
    int4 *dkv_units;
    int4 *sets;  // cleared
};
hipError_t launch_plan_small(const SmallPlan &job, hipStream_t st);
hipError_t launch_plan_ranges(const int32_t *S, const int32_t *N, const int32_t *r,
                              const int32_t *cut, int32_t K, int32_t BM, int32_t BN,
                              int32_t max_q_rows, int32_t max_k_rows, int32_t *q_begin,
                              int32_t *q_len, int32_t *kv_len, int32_t *cu_q, int32_t *cu_k,
                              int32_t *shares_kv, int32_t *fwd_off, int32_t *dkv_off,
                              int32_t cap_fwd, int32_t cap_dkv, int32_t bn_alt, int32_t kv_heads,
                              int32_t compute_units, PlanTotals *totals, hipStream_t st);
// `cost_bound`: no work item costs more (host's bound from the longest sequence); lists whose
// upper bound of items exceeds the rank sort's limit are radix sorted and need
// plan_radix_ints(...) ints of scratch at `radix_hist`
hipError_t launch_plan_items(const skrull_attn_plan_t *p, const int32_t *fwd_off,
                             const int32_t *dkv_off, int32_t cap_fwd, int32_t cap_dkv,
                             int32_t *scratch_fwd, int32_t *scratch_dkv, int32_t *radix_hist,
                             int32_t cost_bound, int32_t compute_units, PlanTotals *totals, hipStream_t st);
// after launch_plan_items: how dK/dV items are shared (`asked`: the caller's head split, 0: the library's own) and the lists of work units
hipError_t launch_plan_units(const skrull_attn_plan_t *p, int32_t asked, int32_t longest_seq, int32_t cap_fwd, int32_t cap_dkv,
                             int32_t compute_units, PlanTotals *totals, hipStream_t st);
int64_t plan_dkv_unit_ints(const skrull_attn_plan_t *p, int32_t asked, int32_t cap_dkv);  // room for dkv_units; 0: no list
int64_t plan_unit_ints(const skrull_attn_plan_t *p, int32_t cap_fwd, int which);  // room for units[which]; 0: no list
int64_t plan_radix_ints(int32_t cap_fwd, int32_t cap_dkv, int32_t cost_bound);

// fwd.hip / bwd.hip
// `trace` (may be null): room for one WgTrace per workgroup of every kernel launched, in
// launch order (launch_bwd: dQ's records, then dK/dV's); grid sizes from the functions below
hipError_t launch_fwd(const skrull_attn_plan_t *p, const void *q, const void *k, const void *v,
                      void *o, float *lse, hipStream_t st, WgTrace *trace);
hipError_t launch_bwd(const skrull_attn_plan_t *p, const void *q, const void *k, const void *v,
                      const void *o, const float *lse, const void *d_o, void *dq, void *dk,
                      void *dv, float *delta, hipStream_t st, hipEvent_t *ev, WgTrace *trace);
int grid_fwd(const skrull_attn_plan_t *p);
int grid_dq(const skrull_attn_plan_t *p);
int grid_dkv(const skrull_attn_plan_t *p);

// probe.hip
hipError_t run_mfma_probe(int blocks, int iters, float *scratch, hipStream_t st, float *ms);
