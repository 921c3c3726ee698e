// Host side of the C ABI: argument validation, plan construction, launches.
// No arithmetic of the method happens here: the descriptor, the work lists, their costs
// and all attention math are produced by kernels (plan.hip, fwd.hip, bwd.hip).  What the
// host derives from the lengths are upper bounds only (how many work items there can be at
// most, for the allocations and grids) and the tuning choices documented in the header,
// which it takes from the totals that the plan kernels return.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <new>

#include "common.h"
#include "skrull_dacp.h"

namespace {

thread_local char g_err[256] = "";

int hip_fail(hipError_t e, const char *what)
{
    snprintf(g_err, sizeof g_err, "%s: %s", what, hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? SKRULL_ENOMEM : SKRULL_EHIP;
}

#define HIP_TRY(expr)                                   \
    do {                                                \
        hipError_t e_ = (expr);                         \
        if (e_ != hipSuccess) { rc = hip_fail(e_, #expr); goto done; } \
    } while (0)

inline bool misaligned(const void *p) { return p == nullptr || ((uintptr_t)p & 15u) != 0; }

inline int64_t align4(int64_t n) { return (n + 3) & ~(int64_t)3; }

// Opt-in kernel timing, per calling thread: events 0/1 bracket the forward kernel, 2..4
// delimit the backward kernels.  A thread that never enables it owns nothing.
struct ProfileState {
    bool on = false, made = false, fwd_seen = false, bwd_seen = false;
    hipEvent_t ev[6];
};
thread_local ProfileState g_prof;

// Opt-in per-workgroup trace, per calling thread: a caller-owned device buffer of WgTrace records.
struct TraceState {
    WgTrace *buf = nullptr;
    size_t records = 0;
};
thread_local TraceState g_trace;

constexpr int32_t kMaxItems = 1 << 20;  // per list (lists above 2,048 items are radix sorted)

// Workspace of skrull_attn_bwd_static, the backward entry point for callers that cannot
// allocate: one array per GPU that the library runs on, held until the process ends.
// In host code the array's name is only a stand-in for the symbol; the device address
// comes from hipGetSymbolAddress, once per device, and is what the kernels are given.
static __device__ __align__(256) unsigned char scratch[SKRULL_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
std::atomic<void *> g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on device `dev`, which must be the current device.
int resolve_scratch(int dev, void **out)
{
    if (dev < 0 || dev >= kMaxDevices) return SKRULL_EUNSUPPORTED;
    void *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev].store(p, std::memory_order_release);  // (a second thread stores the same address)
    }
    *out = p;
    return SKRULL_OK;
}

// Pinned host memory through which a plan's kernels get their input and give its totals back: a few
// slots for the whole process, one for the time of a call; a call that finds none copies instead.  A call that
// cannot wait for its kernels keeps its slot for good: they may still use it.  The memory is asked for as coherent:
// without that the environment (HIP_HOST_COHERENT) decides.
struct PinnedSlots {
    static constexpr int kSlots = 16;
    // Sequences whose description a slot has room for; a longer one is copied.  (600 sequences, 1,128 and 1,982 items:
    // the call takes 147 us with its input and totals copied, 136 through a slot; 1,500 sequences: 390 and 359.)
    static constexpr int32_t kSeqs = 2048;
    static constexpr size_t kIn = 4 * (size_t)kSeqs * sizeof(int32_t), kBytes = (kIn + sizeof(PlanTotals) + 255) & ~(size_t)255;
    std::mutex made;
    unsigned char *base = nullptr;  // held until the process ends
    std::atomic<uint32_t> used{0};

    int32_t *take()
    {
        unsigned char *memory;
        {
            std::lock_guard<std::mutex> lock(made);
            if (!base) {  // (a call that was refused it, for instance beside another thread's capture, leaves it to a later one)
                void *p = nullptr;
                if (hipHostMalloc(&p, kSlots * kBytes, hipHostMallocPortable | hipHostMallocCoherent) == hipSuccess) base = (unsigned char *)p;
                else (void)hipGetLastError();
            }
            memory = base;
        }
        uint32_t u = used.load(std::memory_order_relaxed);
        while (memory) {
            const int free_slot = __builtin_ffs(~u & ((1u << kSlots) - 1)) - 1;
            if (free_slot < 0) break;
            if (used.compare_exchange_weak(u, u | 1u << free_slot, std::memory_order_acquire)) return (int32_t *)(memory + free_slot * kBytes);
        }
        return nullptr;
    }
    void give_back(int32_t *slot)
    {
        if (slot) used.fetch_and(~(1u << (((unsigned char *)slot - base) / kBytes)), std::memory_order_release);
    }
};
PinnedSlots g_pinned;

int check_device(int *dev_out, int *compute_units)
{
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || n < 1) {
        (void)hipGetLastError();
        return SKRULL_EUNSUPPORTED;
    }
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return SKRULL_EUNSUPPORTED;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return SKRULL_EUNSUPPORTED;
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) return SKRULL_EUNSUPPORTED;
    *dev_out = dev;
    *compute_units = prop.multiProcessorCount;
    return SKRULL_OK;
}

// Whether nothing that was queued on `st` so far can run any more.  (A wait ends a capture as invalid: what
// was captured never runs.)
bool is_idle(hipStream_t st)
{
    if (hipStreamSynchronize(st) == hipSuccess) return true;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(st, &capture) == hipSuccess && capture == hipStreamCaptureStatusInvalidated;
}

// A plan's arrays live on the device it was made on: the calls that use them must run there.
int check_plan_device(const skrull_attn_plan_t *plan)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != plan->device) {
        snprintf(g_err, sizeof g_err, "plan was made on device %d, current device is %d", plan->device, dev);
        return SKRULL_EINVAL;
    }
    return SKRULL_OK;
}

}  // namespace

extern "C" {

int skrull_attn_plan(const skrull_attn_problem_t *p, void *hip_stream, skrull_attn_plan_t **out)
{
    if (!p || !out || !p->seq_len || !p->shard_degree || !p->shard_index) return SKRULL_EINVAL;
    const int32_t K = p->num_seqs;
    if (K < 1) return SKRULL_EINVAL;
    if (p->num_q_heads < 1 || p->num_kv_heads < 1 || p->num_q_heads % p->num_kv_heads != 0)
        return SKRULL_EINVAL;
    if (p->head_dim != 64 && p->head_dim != 128) return SKRULL_EINVAL;
    if (!(p->softmax_scale > 0.0f) || !isfinite(p->softmax_scale)) return SKRULL_EINVAL;
    const int32_t BM = p->block_m == 0 ? 256 : p->block_m;
    int32_t BN = p->block_n == 0 ? 128 : p->block_n;  // (left open: may become 192 below)
    if ((BM != 64 && BM != 128 && BM != 256) || (BN != 64 && BN != 128 && BN != 192 && BN != 256))
        return SKRULL_EINVAL;
    const int32_t group = p->num_q_heads / p->num_kv_heads;
    if (p->head_split < 0 || p->head_split > group) return SKRULL_EINVAL;
    if (p->wg_query_rows != 0 && p->wg_query_rows != 128 && p->wg_query_rows != 256) return SKRULL_EINVAL;
    // Entry checks are done here so that they work without a device; the kernel repeats
    // them next to the range computation.  The same pass bounds the number of work
    // items from above (chunk lengths differ by at most one row; a prefix is no longer
    // than its sequence), which sizes the allocations and the grids, so that the whole
    // plan is built with one synchronisation.
    int64_t n_seg = 0;  // query segments: a two-chunk cut contributes two
    int32_t longest_seq = 0;
    const int64_t q_row_bytes = (int64_t)p->num_q_heads * p->head_dim * 2;
    const int64_t kv_row_bytes = (int64_t)p->num_kv_heads * p->head_dim * 2;
    int64_t cap_fwd = 0, cap_dkv = 0;
    for (int32_t k = 0; k < K; ++k) {
        const int32_t s = p->seq_len[k], n = p->shard_degree[k], r = p->shard_index[k];
        const int32_t z = p->shard_cut ? p->shard_cut[k] : SKRULL_CUT_CONTIGUOUS;
        if (z != SKRULL_CUT_CONTIGUOUS && z != SKRULL_CUT_TWO_CHUNKS) return SKRULL_EINVAL;
        if (s < 1 || n < 1 || r < 0 || r >= n || (int64_t)n * (1 + z) > s) return SKRULL_EINVAL;
        n_seg += 1 + z;
        longest_seq = s > longest_seq ? s : longest_seq;
        const int64_t chunks = (int64_t)n * (1 + z), longest = (s + chunks - 1) / chunks;
        // The kernels address a tile as a 32-bit byte offset from the first row of its
        // query segment (rows of Hq*d bf16) or of its key/value prefix (rows of Hkv*d
        // bf16), and prefetch up to four 64-row tiles past the end (those read as zero).
        if ((longest + 256) * q_row_bytes > (int64_t)UINT32_MAX ||
            ((int64_t)s + 256) * kv_row_bytes > (int64_t)UINT32_MAX) {
            snprintf(g_err, sizeof g_err, "sequence %d is too long for 32-bit tile offsets", k);
            return SKRULL_EINVAL;
        }
        cap_fwd += (1 + z) * ((longest + BM - 1) / BM);
        cap_dkv += ((int64_t)s + BN - 1) / BN;
    }
    if (n_seg > INT32_MAX / 2) return SKRULL_EINVAL;
    if (cap_fwd > 8 * (int64_t)kMaxItems || cap_dkv > 8 * (int64_t)kMaxItems) return SKRULL_EINVAL;
    int dev = 0, compute_units = 0;
    int rc = check_device(&dev, &compute_units);
    if (rc != SKRULL_OK) return rc;
    {   // set-up for skrull_attn_bwd_static: this device's address of the static workspace
        void *unused = nullptr;
        if ((rc = resolve_scratch(dev, &unused)) != SKRULL_OK) return rc;
    }

    // dK/dV block size when the caller leaves it open.  At head_dim 64 the kernel has a
    // 12-wavefront shape over 192 key rows; with a sequence of 8,192 tokens or more in the
    // micro-batch it was 3-16 % faster than the 8-wavefront shape over 128 on whole sequences
    // and on slices of distributed ones alike (14 query / 2 KV heads; 2 x 8,192 ... 98,304
    // tokens, both cuts, the benchmark length mixes).  On shorter sequences it wins (7-14 %)
    // exactly where the work list is so short that the heads are split anyway (longest
    // chain above an even share of 128-key items, see head_split below), and loses 2-25 %
    // where it is not: there the fewer, larger workgroups and the split they then need
    // cost more than the third wavefront per SIMD brings.  That second case is decided by the
    // ranges kernel from the costs of the 128-key work list (bn_alt), and comes back in totals.
    int32_t bn_alt = 0;
    if (p->block_n == 0 && p->head_dim == 64) {
        if (longest_seq >= 8192) BN = 192;
        else bn_alt = 192;
    }
    // (cap_dkv counts items of BN key rows; the alternative is larger, so it needs fewer)

    hipStream_t st = (hipStream_t)hip_stream;
    skrull_attn_plan_t *plan = nullptr;
    int32_t *tmp = nullptr, *host_in = nullptr, *pinned = nullptr;
    PlanTotals totals, *totals_h = nullptr;
    int64_t in_stride = 0;
    bool small = false;  // made by one workgroup
    bool queued = false; // kernels have been launched that read and write the slot
    // tmp (released before return): S, N, R, cut [K each] | fwd_off, dkv_off [n_seg+1 each] |
    // totals | unsorted items; a small plan needs none
    const int64_t kin = align4(K), kpad = align4(n_seg + 1);
    const int64_t totals_ints = align4((int64_t)((sizeof(PlanTotals) + 3) / 4));
    // no work item costs more than this many blocks (64 rows is the smallest block; a two-chunk
    // cut adds the query blocks of both chunks)
    const int32_t cost_bound = 2 * (longest_seq / 64 + 2);
    const int64_t radix_ints = plan_radix_ints((int32_t)cap_fwd, (int32_t)cap_dkv, cost_bound);
    const int64_t tmp_ints = 4 * kin + 2 * kpad + totals_ints + 4 * (cap_fwd + cap_dkv) + radix_ints;
    const int64_t desc_ints = 6 * kpad;
    const int64_t queue_ints = SKRULL_QUEUE_INTS * SKRULL_FWD_QUEUE_SLOTS;  // work queues of the forward launches
    const int64_t sets_ints = SKRULL_SETS_INTS;
    int32_t *fwd_off = nullptr, *dkv_off = nullptr, *scratch = nullptr;
    PlanTotals *totals_d = nullptr;
    int64_t unit_ints[SKRULL_UNIT_LISTS] = {}, all_unit_ints = 0, dkv_unit_ints = 0;

    plan = new (std::nothrow) skrull_attn_plan_t();
    if (!plan) return SKRULL_ENOMEM;
    memset(plan, 0, sizeof *plan);
    plan->default_stream = new (std::nothrow) DefaultStream();
    if (!plan->default_stream) { delete plan; return SKRULL_ENOMEM; }
    plan->K = K; plan->NS = (int32_t)n_seg; plan->Hq = p->num_q_heads; plan->Hkv = p->num_kv_heads; plan->d = p->head_dim;
    plan->BM = BM; plan->BN = BN; plan->longest_seq = longest_seq; plan->scale = p->softmax_scale; plan->device = dev;

    pinned = g_pinned.take();
    // One workgroup ranks lists of up to 256 items with two threads or more to an item; above that the several kernels
    // are faster (203 and 354 items: the call takes 61 us by one workgroup, 53 by those; 239 and 420: 66 and 56; 152 and 263: 54
    // and 52; below it 145 and 255: 45 and 50; 109 and 201: 41 and 47).  Where blocks of 192 keys may be taken, a list of
    // such items is two thirds of cap_dkv (167 and 215 items: 46 and 53; 188 and 233: 50 and 55).
    small = pinned && K <= SKRULL_SMALL_PLAN && n_seg <= SKRULL_SMALL_PLAN && cap_fwd <= 256 && cap_dkv <= (bn_alt ? 384 : 256);
    static_assert(384 <= SKRULL_SMALL_PLAN, "a thread to an item");
    in_stride = kin;
    host_in = pinned && K <= PinnedSlots::kSeqs ? pinned : (int32_t *)calloc((size_t)(4 * kin), sizeof(int32_t));
    if (!host_in) { rc = SKRULL_ENOMEM; goto done; }
    memcpy(host_in, p->seq_len, (size_t)K * 4);
    memcpy(host_in + in_stride, p->shard_degree, (size_t)K * 4);
    memcpy(host_in + 2 * in_stride, p->shard_index, (size_t)K * 4);
    if (p->shard_cut) memcpy(host_in + 3 * in_stride, p->shard_cut, (size_t)K * 4);
    else memset(host_in + 3 * in_stride, 0, (size_t)K * 4);

    if (!small) HIP_TRY(hipMalloc((void **)&tmp, (size_t)tmp_ints * sizeof(int32_t)));
    for (int i = 0; i < SKRULL_UNIT_LISTS; ++i) all_unit_ints += unit_ints[i] = plan_unit_ints(plan, (int32_t)cap_fwd, i);
    dkv_unit_ints = plan_dkv_unit_ints(plan, p->head_split, (int32_t)cap_dkv);
    HIP_TRY(hipMalloc((void **)&plan->pool, (size_t)(queue_ints + sets_ints + desc_ints + 4 * (cap_fwd + cap_dkv) + all_unit_ints + dkv_unit_ints) * sizeof(int32_t)));
    plan->fwd_queues = (WorkQueue *)plan->pool;   // (zeroed by the forward calls that use them, before their launch)
    plan->sets = plan->pool + queue_ints;
    plan->cu_q = plan->sets + sets_ints;
    plan->cu_k = plan->cu_q + kpad;
    plan->q_begin = plan->cu_q + 2 * kpad;
    plan->q_len = plan->cu_q + 3 * kpad;
    plan->kv_len = plan->cu_q + 4 * kpad;
    plan->shares_kv = plan->cu_q + 5 * kpad;
    plan->fwd_items = plan->cu_q + desc_ints;
    plan->dkv_items = plan->fwd_items + 4 * cap_fwd;
    {
        int32_t *next = plan->dkv_items + 4 * cap_dkv;
        if (dkv_unit_ints > 0) plan->dkv_units = (int4 *)next;  // (16-byte aligned, as the items are)
        next += dkv_unit_ints;
        for (int i = 0; i < SKRULL_UNIT_LISTS; ++i) {
            if (unit_ints[i] > 0) plan->units[i] = next;
            next += unit_ints[i];
        }
    }
    if (pinned) totals_h = (PlanTotals *)((unsigned char *)pinned + PinnedSlots::kIn);
    queued = true;
    if (small) {
        HIP_TRY(launch_plan_small(SmallPlan{pinned, totals_h, K, (int32_t)in_stride, BM, BN, bn_alt,
                                            INT32_MAX / (p->num_q_heads * p->head_dim), INT32_MAX / (p->num_kv_heads * p->head_dim),
                                            (int32_t)cap_fwd, (int32_t)cap_dkv, p->num_q_heads, p->num_kv_heads, p->head_dim, p->head_split,
                                            longest_seq, compute_units, plan->q_begin, plan->q_len, plan->kv_len, plan->cu_q, plan->cu_k,
                                            plan->shares_kv, plan->fwd_items, plan->dkv_items,
                                            {plan->units[0], plan->units[1], plan->units[2]}, plan->dkv_units,
                                            (int4 *)plan->sets}, st));
    } else {
        fwd_off = tmp + 4 * kin;
        dkv_off = fwd_off + kpad;
        totals_d = (PlanTotals *)(dkv_off + kpad);
        scratch = dkv_off + kpad + totals_ints;
        const int32_t *in = host_in;  // (the kernel reads pinned memory itself)
        if (host_in != pinned) {  // a pageable source is staged by the runtime before the call returns
            HIP_TRY(hipMemcpyAsync(tmp, host_in, (size_t)(4 * kin) * 4, hipMemcpyHostToDevice, st));
            in = tmp;
        }
        HIP_TRY(launch_plan_ranges(in, in + in_stride, in + 2 * in_stride, in + 3 * in_stride, K, BM, BN,
                                   INT32_MAX / (p->num_q_heads * p->head_dim),
                                   INT32_MAX / (p->num_kv_heads * p->head_dim), plan->q_begin,
                                   plan->q_len, plan->kv_len, plan->cu_q, plan->cu_k, plan->shares_kv,
                                   fwd_off, dkv_off, (int32_t)cap_fwd, (int32_t)cap_dkv, bn_alt, p->num_kv_heads,
                                   compute_units, totals_d, st));
        HIP_TRY(launch_plan_items(plan, fwd_off, dkv_off, (int32_t)cap_fwd, (int32_t)cap_dkv, scratch,
                                  scratch + 4 * cap_fwd, scratch + 4 * (cap_fwd + cap_dkv), cost_bound, compute_units,
                                  totals_d, st));
        HIP_TRY(launch_plan_units(plan, p->head_split, longest_seq, (int32_t)cap_fwd, (int32_t)cap_dkv, compute_units, totals_d, st));
        HIP_TRY(hipMemcpyAsync(pinned ? totals_h : &totals, totals_d, sizeof totals, hipMemcpyDeviceToHost, st));
    }
    HIP_TRY(hipStreamSynchronize(st));
    queued = false;
    if (pinned) memcpy(&totals, totals_h, sizeof totals);
    if (totals.bad_entry != 0 || totals.n_seg != plan->NS || totals.total_q > INT32_MAX ||
        totals.total_k > INT32_MAX || totals.n_fwd > kMaxItems || totals.n_dkv > kMaxItems ||
        totals.n_fwd > cap_fwd || totals.n_dkv > cap_dkv) {
        snprintf(g_err, sizeof g_err, "micro-batch too large or invalid entry %d", totals.bad_entry - 1);
        rc = SKRULL_EINVAL;
        goto done;
    }
    if (totals.block_n != BN && totals.block_n != bn_alt) { rc = SKRULL_EHIP; snprintf(g_err, sizeof g_err, "plan kernels returned block_n %d", totals.block_n); goto done; }
    plan->BN = totals.block_n;
    plan->total_q = (int32_t)totals.total_q;
    plan->total_k = (int32_t)totals.total_k;
    plan->n_fwd = (int32_t)totals.n_fwd;
    plan->n_dkv = (int32_t)totals.n_dkv;
    plan->pairs = totals.pairs;
    for (int i = 0; i < SKRULL_UNIT_LISTS; ++i) plan->n_units[i] = totals.n_units[i];
    // Workgroup shape of the forward and dQ kernels.  Several 4-wavefront workgroups per compute
    // unit hide each other's start-up, drain and barriers, but they also stretch each other's
    // work items (three share a unit and its oldest wave is served first), and a launch ends only
    // when its last stretched item does; so the small shape pays once the launch holds enough
    // work to bury that tail: at head_dim 64 from 24 blocks of 256 query rows x heads per compute unit or
    // 1.5e9 attended (query, key, head) triples on, at head_dim 128 (forward only: the small dQ shape
    // does not fit the LDS twice) from 16 such blocks on while no sequence exceeds 8,192 tokens, where the
    // 8-wavefront workgroup's deeper tile ring and halved tile traffic take over.  Measured on 8 to 64
    // query heads x 16,384 to 32,768 tokens x sequences of 256 to 32,768 tokens (profiles/shape_sweep_wg.txt):
    // where this picks it the small forward is 4-15 % faster at head_dim 64 (dQ within 1.6 %) and up to 10 %
    // at 128, 0.3 % slower at worst; where it does not, the small dQ loses up to 25 % at head_dim 64 while
    // the small forward is between 14 % faster and 5 % slower (one choice serves both), and at 128 the
    // forward is between 9 % faster (few heads) and 3 % slower.  Forward and dQ together: 0.6 % behind the better
    // shape on average, 7 % at worst.
    if (p->wg_query_rows != 0) {
        plan->wg_query_rows = p->wg_query_rows;
    } else {
        const double blocks_per_cu = (double)plan->Hq * (double)totals.total_q / (256.0 * (double)compute_units);
        const double triples = (double)totals.pairs * (double)plan->Hq;
        const bool small_shape = p->head_dim == 64 ? (blocks_per_cu >= 24.0 || triples >= 1.5e9)
                                                   : (longest_seq <= 8192 && blocks_per_cu >= 16.0);
        plan->wg_query_rows = small_shape ? 128 : 256;
    }
    // At head_dim 64, where the library chooses and has not taken the small shape:
    //  Both kernels also have a shape of 12 wavefronts to a workgroup, three per SIMD, which share the tiles of
    //    keys that two per SIMD would wait for.  Each wavefront runs slower, so the longest unit must not be what
    //    the launch waits for, and its row blocks must fill 12 about as well as 8 (they do not with one head per group).
    //    Against 8 wavefronts, by r = the longest unit / an even share per compute unit, on 28 micro-batches of 14/2 heads
    //    (forward) and 40 more (backward): forward 2 to 8 % less time up to r = 0.89, 6 % more at 0.91, 8 % less at 0.95, 15
    //    to 30 % more from 1.1 on; backward 1 to 5 % less up to 0.95, 4 to 10 % more from 1.08 on.  On 54 forwards of 9 to 48
    //    heads, by what 12 leave empty beside 8: 5 to 15 % less up to 16 % (24/8 heads, 8,192 tokens
    //    of 8 to 511: 33.5 -> 28.4 us), between 6 % less and 1 % more at 30 % (two heads per group).
    //  A launch whose workgroups of 4 wavefronts, one per 128 rows and head, all run at once has those: half as
    //    many wavefronts share a unit, where most of the chip would stay idle beside them.  Measured on 40 micro-batches of 16
    //    to 6,000 tokens, 4 to 16 heads: forward up to 20 % less time (7 to 10 % in the middle, 2 % more at worst), backward 4
    //    to 7 % less; a third more than fits, and dQ lost 11 to 43 %.
    //    Not where those of 8 all run at once too and either end with units of up to 128 rows, that is, of four wavefronts in any case (384
    //    tokens, 4/4 heads: forward and dQ 26.7 us with 8, 30.5 with 4), and the next longest ones are enough shorter, or are many and
    //    short, where starts count (64 of 200, 4/4 heads: 31.8 and 34.3).  677 launches of eight head shapes against 8 wavefronts: forward and dQ
    //    together 0.929 of the time, 1.146 at worst, with 4 throughout; 0.927 and 1.033 this way.
    //  A forward of which workgroups of 4 all run at once only because short items leave some of them without rows has those too: 5 to
    //    31 % less time than with 8 on 13 forwards of 498 to 768 of them, 0 to 56 % less on 24 of thirteen kinds of heads with 800 to 7,200 tokens; a few
    //    more than fit (three to a compute unit), and it takes up to 50 % more.
    plan->fwd_waves = plan->wg_query_rows / 32;
    plan->dq_waves = plan->d == 64 ? plan->wg_query_rows / 32 : 8;
    if (p->wg_query_rows == 0 && plan->wg_query_rows == 256 && plan->d == 64) {
        if (plan->units[2] && group > 1 && 5 * 12 * (int64_t)plan->n_units[2] <= 6 * 8 * (int64_t)plan->n_units[1] &&
            10 * (int64_t)totals.fwd_longest * compute_units <= 9 * totals.fwd_load * plan->Hkv)
            plan->fwd_waves = plan->dq_waves = 12;
        else if (2 * totals.n_fwd * plan->Hq <= 3 * (int64_t)compute_units) {
            const int64_t of_eight = (int64_t)plan->n_units[1] * plan->Hkv;
            const int32_t longest = totals.fwd_longest - 16, full = totals.fwd_longest_full - 16;
            const bool once = plan->units[2] && of_eight <= compute_units, many = 2 * of_eight >= compute_units;
            const bool ends_small = full > 0 && (4 * full <= 3 * longest || (many && 5 * full <= 4 * longest + 4));
            if (!(once && (ends_small || (longest <= 8 && many)))) plan->dq_waves = plan->fwd_waves = 4;
        } else if (plan->units[0] && (int64_t)plan->n_units[0] * plan->Hkv <= 3 * (int64_t)compute_units) {
            plan->fwd_waves = 4;
        }
    }
    // At head_dim 128, where the library chooses and has not taken the small shape, the forward has it by itself
    //  for lists without long sequences from 6 blocks of 256 query rows x heads per compute unit on, where starts and ends of
    //    units are most of the time and the second workgroup of a unit hides them: against 8 wavefronts 0 to 8 % less time (65
    //    forwards, 4 % on average); from 4 to 6 blocks 5 % less to 6 % more, with sequences of 2,049 to 4,096 tokens within 3 % from 8 blocks
    //    on, with longer ones up to 3 % more;
    //  where 8 wavefronts would run at once: 7 % less time on 128 forwards, 17 at best, 2 % more at worst; but not where the longest sequence
    //    has 257 to 384 tokens, whose last block is four wavefronts in any case (8 % more to 2 % less).
    if (p->wg_query_rows == 0 && plan->wg_query_rows == 256 && plan->d == 128) {
        const double blocks_per_cu = (double)plan->Hq * (double)totals.total_q / (256.0 * (double)compute_units);
        const bool at_once = (int64_t)totals.n_fwd * plan->Hq <= compute_units || (plan->units[1] && (int64_t)plan->n_units[1] * plan->Hkv <= compute_units);
        if ((longest_seq <= 2048 && blocks_per_cu >= 6.0) || (at_once && (longest_seq <= 256 || longest_seq > 384))) plan->fwd_waves = 4;
    }
    // Of dQ workgroups of 4 three share a compute unit, each slower than one of the two that the pipelined kernel has
    // there.  Measured on 173 micro-batches, of 4 to 16 heads and 8 to 7,516 units, pipelined against not:
    //  up to two units per compute unit all run at once either way, and a unit is faster pipelined once it is long
    //    enough: from 24 half tiles of keys on (fwd_longest counts 16 for a unit's start and end) 1 to 12 % less time (all
    //    of 63; 2 % at 24 to 31, 10 % from 130 on), at 20 to 23 from 5 % less to 1 % more, below that 1 % more on average, 8 at worst;
    //  up to three per compute unit the pipelined kernel has a second round: 2 to 21 % more (all of 11);
    //  above that by r = the longest unit / an even share per place: up to r = 1 it takes as much or up to 6 % more
    //    (40 of 41, the other 1 % less), from 1.3 on, where a round of long units is what the launch waits for, 7 to 16 % less.
    plan->dq_piped = false;
    if (plan->dq_waves == 4 && plan->units[2]) {
        const double places = 3.0 * (double)compute_units, units = (double)plan->n_units[0] * (double)plan->Hkv;
        const double share = (double)totals.fwd_load * (double)plan->n_units[0] / (double)(plan->n_units[2] > 0 ? plan->n_units[2] : 1) * (double)plan->Hkv / places;
        if (units <= 2.0 * (double)compute_units) plan->dq_piped = totals.fwd_longest >= 40;
        else if (units > places) plan->dq_piped = (double)totals.fwd_longest >= share;
    }
    // In one launch with dK/dV of 12 wavefronts, dQ in units of 12 row blocks against the units above, 66 backwards of 14/2
    // heads: where those are for 8 wavefronts 2 to 11 % less time (all of 14), for 4 that are not pipelined up to 13 % less (10 of 10; 2 % more at
    // worst), for 4 pipelined 5 to 20 % less with sequences of up to 2,500 tokens, within 2 % at 4,300 and 4,700, 5 to 18 % more
    // from 10,000 on (a slice's prefix counts).  With other groups, 80 backwards of 300 to 30,000 tokens: of 2 as long on average (8 % less to
    // 5 % more), of 3 and 8 3 % less (14 % to 0), of 4, 5 and 7 1 to 2 % less (8 % to 1 % more), of 16 as long (within 2 %).  One head per group does not fill 12 from a sequence's last blocks.
    plan->dq_packed = plan->d == 64 && group > 1 && plan->units[2] && (plan->dq_waves == 8 || (plan->dq_waves == 4 && (!plan->dq_piped || totals.fwd_longest <= 128 + 16)));
    plan->head_split = totals.split.head_split;
    plan->n_split = totals.split.n_split;
    plan->n_whole_first = totals.split.n_whole_first;
    plan->split_parts = totals.split.parts;
    plan->split_chain = totals.split.chain;
    plan->split_compact = totals.split.compact;
    plan->n_dkv_units = totals.n_dkv_units;
    rc = SKRULL_OK;
done:
    if (host_in != pinned) free(host_in);
    if (pinned && (!queued || is_idle(st))) g_pinned.give_back(pinned);  // (else nobody may have it any more)
    if (tmp) (void)hipFree(tmp);
    if (rc != SKRULL_OK) {
        if (plan) {
            if (plan->pool) (void)hipFree(plan->pool);
            delete plan->default_stream;
            delete plan;
        }
        return rc;
    }
    *out = plan;
    return SKRULL_OK;
}

int skrull_attn_plan_info(const skrull_attn_plan_t *plan, skrull_attn_plan_info_t *info)
{
    if (!plan || !info) return SKRULL_EINVAL;
    info->num_seqs = plan->K;
    info->num_q_heads = plan->Hq;
    info->num_kv_heads = plan->Hkv;
    info->head_dim = plan->d;
    info->block_m = plan->BM;
    info->block_n = plan->BN;
    info->total_q = plan->total_q;
    info->total_k = plan->total_k;
    info->n_fwd_items = plan->n_fwd;
    info->n_dkv_items = plan->n_dkv;
    info->attended_pairs = plan->pairs;
    info->useful_flops_fwd = 4 * plan->pairs * plan->d * plan->Hq;
    info->useful_flops_bwd = 10 * plan->pairs * plan->d * plan->Hq;
    info->bwd_workspace_bytes = base_workspace(plan->Hq, plan->total_q);
    if (plan->head_split > 1)  // fp32 partial dK and dV of every share of the heads
        info->bwd_workspace_bytes += 2 * (int64_t)plan->head_split * plan->total_k * plan->Hkv * plan->d * 4;
    else
        info->bwd_workspace_bytes += partial_bytes(SplitChoice{plan->head_split, plan->n_split, plan->n_whole_first, plan->split_parts, plan->split_chain, plan->split_compact},
                                                   plan->BN, plan->total_k, plan->Hkv, plan->d);
    info->num_segments = plan->NS;
    info->head_split = plan->head_split;
    info->wg_query_rows = plan->wg_query_rows;
    info->shapes = plan->fwd_waves | plan->dq_waves << 8 | (plan->dq_waves == 8 || plan->dq_piped ? 1 << 16 : 0);
    return SKRULL_OK;
}

int skrull_attn_plan_export(const skrull_attn_plan_t *plan, int which, void *dst, size_t bytes)
{
    if (!plan || !dst) return SKRULL_EINVAL;
    const int32_t *src = nullptr;
    size_t n = 0;
    switch (which) {
    case SKRULL_ARRAY_CU_Q: src = plan->cu_q; n = (size_t)plan->NS + 1; break;
    case SKRULL_ARRAY_CU_K: src = plan->cu_k; n = (size_t)plan->NS + 1; break;
    case SKRULL_ARRAY_Q_BEGIN: src = plan->q_begin; n = (size_t)plan->NS; break;
    case SKRULL_ARRAY_Q_LEN: src = plan->q_len; n = (size_t)plan->NS; break;
    case SKRULL_ARRAY_KV_LEN: src = plan->kv_len; n = (size_t)plan->NS; break;
    case SKRULL_ARRAY_SHARES_KV: src = plan->shares_kv; n = (size_t)plan->NS; break;
    case SKRULL_ARRAY_FWD_ITEMS: src = plan->fwd_items; n = (size_t)plan->n_fwd * 4; break;
    case SKRULL_ARRAY_DKV_ITEMS: src = plan->dkv_items; n = (size_t)plan->n_dkv * 4; break;
    default: return SKRULL_EINVAL;
    }
    if (bytes != n * sizeof(int32_t)) return SKRULL_EINVAL;
    if (int rc = check_plan_device(plan)) return rc;
    hipError_t e = hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpy(export)");
    return SKRULL_OK;
}

int skrull_attn_fwd(const skrull_attn_plan_t *plan, const void *q, const void *k, const void *v,
                    void *o, float *lse, void *hip_stream)
{
    if (!plan) return SKRULL_EINVAL;
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(o) || misaligned(lse))
        return SKRULL_EINVAL;
    if (int rc = check_plan_device(plan)) return rc;
    if (g_prof.on) (void)hipEventRecord(g_prof.ev[0], (hipStream_t)hip_stream);
    WgTrace *trace = nullptr;
    if (g_trace.buf) {
        if ((size_t)grid_fwd(plan) > g_trace.records) return SKRULL_EINVAL;
        trace = g_trace.buf;
    }
    hipError_t e = launch_fwd(plan, q, k, v, o, lse, (hipStream_t)hip_stream, trace);
    if (e != hipSuccess) return hip_fail(e, "forward launch");
    if (g_prof.on) { (void)hipEventRecord(g_prof.ev[1], (hipStream_t)hip_stream); g_prof.fwd_seen = true; }
    return SKRULL_OK;
}

int skrull_attn_bwd(const skrull_attn_plan_t *plan, const void *q, const void *k, const void *v,
                    const void *o, const float *lse, const void *d_o, void *dq, void *dk, void *dv,
                    void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!plan) return SKRULL_EINVAL;
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(o) || misaligned(lse) ||
        misaligned(d_o) || misaligned(dq) || misaligned(dk) || misaligned(dv) ||
        misaligned(workspace))
        return SKRULL_EINVAL;
    skrull_attn_plan_info_t info;
    skrull_attn_plan_info(plan, &info);
    if ((int64_t)workspace_bytes < info.bwd_workspace_bytes) return SKRULL_EINVAL;
    if (int rc = check_plan_device(plan)) return rc;
    WgTrace *trace = nullptr;
    if (g_trace.buf) {  // after the forward's records
        const size_t first = (size_t)grid_fwd(plan);
        if (first + grid_dq(plan) + grid_dkv(plan) > g_trace.records) return SKRULL_EINVAL;
        trace = g_trace.buf + first;
    }
    hipError_t e = launch_bwd(plan, q, k, v, o, lse, d_o, dq, dk, dv, (float *)workspace,
                              (hipStream_t)hip_stream, g_prof.on ? g_prof.ev + 2 : nullptr, trace);
    if (e != hipSuccess) return hip_fail(e, "backward launch");
    if (g_prof.on) g_prof.bwd_seen = true;
    return SKRULL_OK;
}

int skrull_attn_bwd_static(const skrull_attn_plan_t *plan, const void *q, const void *k, const void *v,
                           const void *o, const float *lse, const void *d_o, void *dq, void *dk,
                           void *dv, void *hip_stream)
{
    if (!plan) return SKRULL_EINVAL;
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(o) || misaligned(lse) ||
        misaligned(d_o) || misaligned(dq) || misaligned(dk) || misaligned(dv))
        return SKRULL_EINVAL;
    skrull_attn_plan_info_t info;
    skrull_attn_plan_info(plan, &info);
    if (info.bwd_workspace_bytes > (int64_t)SKRULL_STATIC_SCRATCH_BYTES) {
        snprintf(g_err, sizeof g_err,
                 "this plan needs %lld bytes of backward workspace, the static one holds %lld "
                 "(use skrull_attn_bwd, or a plan with head_split = 1 if the partial sums are what is large)",
                 (long long)info.bwd_workspace_bytes, (long long)SKRULL_STATIC_SCRATCH_BYTES);
        return SKRULL_EINVAL;
    }
    if (int rc = check_plan_device(plan)) return rc;
    void *ws = nullptr;  // resolved when the plan was made; looked up again only if that was another process state
    if (int rc = resolve_scratch(plan->device, &ws)) return rc;
    hipError_t e = launch_bwd(plan, q, k, v, o, lse, d_o, dq, dk, dv, (float *)ws,
                              (hipStream_t)hip_stream, g_prof.on ? g_prof.ev + 2 : nullptr, nullptr);
    if (e != hipSuccess) return hip_fail(e, "backward launch");
    if (g_prof.on) g_prof.bwd_seen = true;
    return SKRULL_OK;
}

void skrull_attn_plan_destroy(skrull_attn_plan_t *plan)
{
    if (!plan) return;
    if (plan->pool) (void)hipFree(plan->pool);
    delete plan->default_stream;
    delete plan;
}

int skrull_attn_mfma_ceiling(void *hip_stream, float *tflops)
{
    if (!tflops) return SKRULL_EINVAL;
    int dev = 0, compute_units = 0;
    int rc = check_device(&dev, &compute_units);
    if (rc != SKRULL_OK) return rc;
    const int blocks = compute_units, iters = 40000;  // ~20 ms of MFMAs
    float ms = 0.0f;
    void *ws = nullptr;  // the probe's sink (blocks x 2 KB) is the static workspace: nothing is allocated
    if ((size_t)blocks * 512 * sizeof(float) > (size_t)SKRULL_STATIC_SCRATCH_BYTES) return SKRULL_EUNSUPPORTED;
    if ((rc = resolve_scratch(dev, &ws)) != SKRULL_OK) return rc;
    hipError_t e = run_mfma_probe(blocks, iters, (float *)ws, (hipStream_t)hip_stream, &ms);
    if (e != hipSuccess) return hip_fail(e, "MFMA probe");
    // blocks x 8 waves x iters x 4 MFMAs x 32*32*16*2 flop
    *tflops = (float)((double)blocks * 8.0 * iters * 4.0 * 32768.0 / (ms * 1e-3) / 1e12);
    return SKRULL_OK;
}

int skrull_attn_trace(void *records, size_t bytes)
{
    if (records && (misaligned(records) || bytes < sizeof(WgTrace))) return SKRULL_EINVAL;
    g_trace.buf = (WgTrace *)records;
    g_trace.records = records ? bytes / sizeof(WgTrace) : 0;
    return SKRULL_OK;
}

int skrull_attn_trace_layout(const skrull_attn_plan_t *plan, int32_t first_record[3], int32_t num_records[3])
{
    if (!plan || !first_record || !num_records) return SKRULL_EINVAL;
    num_records[0] = grid_fwd(plan);
    num_records[1] = grid_dq(plan);
    num_records[2] = grid_dkv(plan);
    first_record[0] = 0;
    first_record[1] = num_records[0];
    first_record[2] = num_records[0] + num_records[1];
    return SKRULL_OK;
}

int skrull_attn_profile(int enable)
{
    ProfileState &ps = g_prof;
    if (enable && !ps.made) {
        for (int i = 0; i < 6; ++i) {
            hipError_t e = hipEventCreate(&ps.ev[i]);
            if (e != hipSuccess) {
                while (i-- > 0) (void)hipEventDestroy(ps.ev[i]);
                return hip_fail(e, "hipEventCreate");
            }
        }
        ps.made = true;
    }
    if (!enable && ps.made) {  // switching off releases the thread's events
        for (int i = 0; i < 6; ++i) (void)hipEventDestroy(ps.ev[i]);
        ps.made = false;
    }
    ps.on = enable != 0;
    ps.fwd_seen = ps.bwd_seen = false;
    return SKRULL_OK;
}

int skrull_attn_profile_read(float ms[4])
{
    ProfileState &ps = g_prof;
    if (!ms || !ps.on) return SKRULL_EINVAL;
    for (int i = 0; i < 4; ++i) ms[i] = -1.0f;
    hipError_t e;
    if (ps.fwd_seen) {
        if ((e = hipEventSynchronize(ps.ev[1])) != hipSuccess) return hip_fail(e, "hipEventSynchronize");
        if ((e = hipEventElapsedTime(&ms[0], ps.ev[0], ps.ev[1])) != hipSuccess) return hip_fail(e, "hipEventElapsedTime");
    }
    if (ps.bwd_seen) {
        // backward events: ev[2] start, ev[3] after dQ (which also forms D), ev[4] after dK/dV
        if ((e = hipEventSynchronize(ps.ev[4])) != hipSuccess) return hip_fail(e, "hipEventSynchronize");
        ms[1] = 0.0f;
        if ((e = hipEventElapsedTime(&ms[3], ps.ev[2], ps.ev[3])) != hipSuccess) return hip_fail(e, "hipEventElapsedTime");
        if ((e = hipEventElapsedTime(&ms[2], ps.ev[3], ps.ev[4])) != hipSuccess) return hip_fail(e, "hipEventElapsedTime");
    }
    return SKRULL_OK;
}

const char *skrull_attn_strerror(int code)
{
    thread_local char buf[320];
    switch (code) {
    case SKRULL_OK: return "ok";
    case SKRULL_EINVAL:
        if (g_err[0]) { snprintf(buf, sizeof buf, "invalid argument (%s)", g_err); return buf; }
        return "invalid argument";
    case SKRULL_ENOMEM: return "out of memory";
    case SKRULL_EHIP: snprintf(buf, sizeof buf, "HIP runtime error (%s)", g_err); return buf;
    case SKRULL_EUNSUPPORTED: return "no gfx950 (MI355X) device available";
    case SKRULL_ESCHED: return "DACP scheduling error: the micro-batch does not fit the buckets";
    default: return "unknown error code";
    }
}

}  // extern "C"
