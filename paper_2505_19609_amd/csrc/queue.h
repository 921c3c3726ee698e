// Work queues of a persistent launch.
//
// The hardware deals the workgroups of a grid to the eight dies (XCDs) round-robin, block b
// to die b mod 8, and only balances the load inside a die.  The dies of one chip do not run
// at one speed (on the measured parts the same list of work items took one die 6 % longer
// than another), so a grid with one workgroup per work item ends with the fast dies idle for
// the last 3-5 % of the launch.  Here a launch instead starts as many workgroups as the chip
// holds at once, and each takes work items until none is left: the one of its block index,
// then from its own die's queue (work items w = die, die + 8, die + 16, ... in list order,
// which keeps the heads of one KV group on one die and its L2, as the static mapping did),
// then from the queue with the most items left.  The work lists are sorted by descending cost, so what is stolen at
// the end are the smallest items: the paper's rule (Alg. 1: the next piece goes to argmin of
// the loads) applied across dies at run time, since their speeds are not known beforehand.
//
// In the forward the longest items, as many as a launch has workgroups ("first items"), carry a mark each that
// says whether they are taken, and a die's first counts, one for each of its first items, stand for any of
// those that has no mark yet.  So a workgroup takes the item of its block index when it starts, but one that
// starts late, for instance because another stream's kernel holds its compute unit, has kept it from nobody.
// (Without marks, with half of the chip held by another launch, the items of the workgroups that had to wait
// began when all the short ones were done: after 310 us of a forward of 24 sequences of 1,500 tokens and
// 600 of 40, 8/8 heads of 128; now all the long ones begin within 65 us.)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

constexpr int kFirstWords = 3;
constexpr int kMaxFirst = 8 * 32 * kFirstWords;  // most first items of a launch
struct WorkQueue {                // of one die
    int32_t next;                 // how many of the die's work items have been handed out
    uint32_t taken[kFirstWords];  // marks of its first items, a bit each
};
// A launch has eight of them, this many apart.  Atomics on one 128-byte line wait for each other, and all
// workgroups of a launch send their first ones together: with the eight queues in one line the forward of 64
// sequences, 26,624 tokens, 14/2 heads of 64, takes 83 us, with a line each 75, and one of 10,573 tokens 45
// and 38.  (The workspace of a backward has room for one line per launch: what calls use that clear their queues first.)
constexpr int kQueueStride = 8, kQueueStrideWorkspace = 1;

// The kernel's one argument (a struct of parameters), read anew through an opaque pointer: in a
// persistent kernel every parameter is an invariant of the work loop, and kept from one work
// item to the next they filled the scalar registers and then, as spilled lanes, vector ones.
template <typename P> using kernarg_t = const P __attribute__((address_space(4))) *;
template <typename P> __device__ __forceinline__ kernarg_t<P> kernarg()
{
    kernarg_t<P> p = (kernarg_t<P>)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// A plan's array, which no kernel that reads it this way writes: read through the scalar cache.
template <typename T> __device__ __forceinline__ T plan_value(const T *array, int i)
{
    return ((const T __attribute__((address_space(4))) *)(uintptr_t)array)[i];
}

// A struct of wave-uniform values, said to be so (a choice between loaded ones and none lands in
// vector registers).
template <typename S> __device__ __forceinline__ S uniform(const S &s)
{
    static_assert(sizeof(S) % 4 == 0, "made of 32-bit words");
    struct W { int w[sizeof(S) / 4]; };
    W w = __builtin_bit_cast(W, s);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(S) / 4); ++i) w.w[i] = __builtin_amdgcn_readfirstlane(w.w[i]);
    return __builtin_bit_cast(S, w);
}

// (The atomics of one lane below take an address and a value that the compiler cannot see to be uniform:
// for uniform ones it combines the lanes that are on, one here, and waits for the answer at once to
// spread it to them.)
__device__ __forceinline__ int opaque(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}
__device__ __forceinline__ int next_count(WorkQueue *q, int stride, int xcd)
{
    return __hip_atomic_fetch_add(&q[(uint32_t)opaque(stride * xcd)].next, opaque(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Marks first item 32 * word + bit of a die; the word's marks before that.
__device__ __forceinline__ uint32_t mark_first(WorkQueue *q, int stride, int xcd, int word, int bit)
{
    return __hip_atomic_fetch_or(&q[(uint32_t)opaque(stride * xcd)].taken[word], (uint32_t)opaque(1 << bit), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The work item that count `k` of die `xcd`'s queue stands for, or kQueueEmpty.
constexpr int kNoWork = -1, kQueueEmpty = -2;
template <bool FIRST> __device__ __forceinline__ int counted_work(WorkQueue *q, int stride, int n_work, int n_first, int xcd, int k)
{
    const int mine = (n_first - xcd + 7) / 8;  // this die's first items
    while (FIRST && __builtin_expect(k < mine, 0)) {
        for (int i = 0; 32 * i < mine;) {
            const uint32_t seen = __hip_atomic_load(&q[stride * xcd].taken[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int bit = __ffs(~seen) - 1;
            if (~seen == 0 || 32 * i + bit >= mine) { ++i; continue; }
            if (!(mark_first(q, stride, xcd, i, bit) >> bit & 1)) return 8 * (32 * i + bit) + xcd;
        }
        // all marked, one by a late workgroup whose own count was past them: that one has two items
        k = next_count(q, stride, xcd);
    }
    const int w = 8 * k + xcd;
    return w < n_work ? w : kQueueEmpty;
}

// The next item of the queue with the most items left; kNoWork when every queue is empty.  Called by
// one lane.  Counters are device-scope atomics (the dies' L2 caches are not coherent with
// each other for plain accesses).
template <bool FIRST> __device__ __forceinline__ int stolen_work(WorkQueue *q, int stride, int n_work, int n_first)
{
    for (;;) {
        int best = -1, best_left = 0;
        for (int y = 0; y < 8; ++y) {
            const int ky = __hip_atomic_load(&q[stride * y].next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int left = (n_work - y + 7) / 8 - ky;  // items of queue y: ceil((n_work - y) / 8)
            if (left > best_left) { best_left = left; best = y; }
        }
        if (best < 0) return kNoWork;
        const int w = counted_work<FIRST>(q, stride, n_work, n_first, best, next_count(q, stride, best));
        if (w >= 0) return w;
        // someone else took its last item in between: look again (every failed attempt
        // means a queue has run empty, so this ends after at most eight rounds)
    }
}

// Die this wave runs on (XCC_ID register, bits 0-3).
__device__ __forceinline__ int my_xcd() { return __builtin_amdgcn_readfirstlane(__builtin_amdgcn_s_getreg((31 << 11) | 20) & 7); }

// The work of a persistent workgroup: one item after another until there is none (kNoWork).  Without a
// queue (q == nullptr) the workgroup does the one item of its block index, as in a plain grid.
// The next item is asked for while the current one still computes: `ask` (one lane sends the
// atomic), `post` (that lane leaves the answer in LDS), a barrier of the caller's, `take`
// (every wave reads it) -- with the claim, its two barriers and the loads of the item's
// descriptor between two items, a workgroup stood still for 3 to 3.5 us per item (a quarter
// of the forward of 64 short sequences, 14/2 heads of 64).  Asked for near the END of an item,
// so that what a workgroup holds back from the others is at most about to start.  `take` says
// kQueueEmpty when the die's own queue is used up: the search of the others (`other`) is left until
// the item's results are stored, because at the end of a launch, when most workgroups search at
// once, it takes up to 20 us and held back the last stores (114 sequences of about 250 tokens, 32/8
// heads of 128: the last items of the forward took 27 us instead of 7).
// With FIRST the first item is the one of the block index, if nobody has taken it.  Blocks go to
// the compute units of a die in turn, so the workgroups that share a unit start with items a third or
// half of the first round apart; with items claimed in order of arrival a unit could start with three of the longest
// (30,934 tokens in 3 sequences, 4/4 heads of 64: forward 547 us claimed, 503 by index).  Where a
// unit holds one workgroup and the items are alike, the order of arrival staggers them a little, and
// they run faster than in step (dK/dV, 27 sequences, 20,011 tokens, 32/8 heads of 128: 3 %).  dQ claims
// too: by index it was as fast at head_dim 128 without marks, but with them 1 to 3 % slower on short lists
// (measured with all counts of a backward in one line, as they are on streams other than the default one).
// `slot` is two ints of LDS; the caller has a barrier between a `take` and the next `post`.
// `Source` says where the queue is (queue(), or null; stride(), its dies' distance) and how many items there are (items()).
template <bool FIRST, typename Source> struct WorkFeed {
    Source src;
    int n_first, pending;  // how many items are first items; the count asked for, or ~ an item
    int *slot;                     // the next item; with FIRST also one more that this workgroup has taken, or -1

    // The first item.  `begin` sends the atomics, so that the loads of its descriptor are under way with
    // them; `first` says which item it is.
    __device__ __forceinline__ uint32_t begin()
    {
        const int b = (int)blockIdx.x;
        uint32_t marks = ~0u;
        if (FIRST && src.queue() && b < n_first && threadIdx.x == 0) {
            pending = next_count(src.queue(), src.stride(), b & 7);
            marks = mark_first(src.queue(), src.stride(), b & 7, b >> 8, b >> 3 & 31);
        }
        return marks;
    }
    __device__ __forceinline__ int first(uint32_t marks)
    {
        const int b = (int)blockIdx.x;
        if (!src.queue()) return b;
        if (FIRST && threadIdx.x == 0) slot[1] = -1;
        if (!FIRST || b >= n_first) return again();
        if (threadIdx.x == 0) {
            const bool own = !(marks >> (b >> 3 & 31) & 1);
            slot[0] = b;
            if (__builtin_expect(!own || pending >= (n_first - (b & 7) + 7) / 8, 0)) {
                // late: another item instead, or, where others had the rights to all first items but had
                // not marked this one, another item as well
                const int w = counted_work<FIRST>(src.queue(), src.stride(), src.items(), n_first, b & 7, pending);
                slot[own ? 1 : 0] = w;
            }
        }
        __syncthreads();
        const int w = take();
        return w == kQueueEmpty ? other() : w;
    }
    __device__ __forceinline__ void ask()
    {
        if (src.queue() && threadIdx.x == 0) {
            const int more = FIRST ? slot[1] : -1;
            if (__builtin_expect(more >= 0, 0)) {
                pending = ~more;
                slot[1] = -1;
            } else {
                pending = next_count(src.queue(), src.stride(), my_xcd());
            }
        }
    }
    __device__ __forceinline__ void post()
    {
        if (src.queue() && threadIdx.x == 0) *slot = FIRST && pending < 0 ? ~pending : counted_work<FIRST>(src.queue(), src.stride(), src.items(), n_first, my_xcd(), pending);
    }
    __device__ __forceinline__ int take() const { return src.queue() ? __builtin_amdgcn_readfirstlane(*slot) : kNoWork; }
    // after kQueueEmpty: an item of another die's queue
    __device__ __forceinline__ int other()
    {
        __syncthreads();  // everyone has read the slot
        if (threadIdx.x == 0) *slot = stolen_work<FIRST>(src.queue(), src.stride(), src.items(), n_first);
        __syncthreads();
        return take();
    }
    // all of it at once, for a workgroup that has no work to hide it behind
    __device__ __forceinline__ int again()
    {
        if (!src.queue()) return kNoWork;
        __syncthreads();  // everyone has read the slot
        ask();
        post();
        __syncthreads();
        const int w = take();
        return w == kQueueEmpty ? other() : w;
    }
};

// Zeroes what a later launch's workgroups will share; by the threads of one workgroup.
__device__ __forceinline__ void clear_state(int32_t *state, int ints)
{
    for (int i = threadIdx.x; i < ints / 4; i += blockDim.x) ((int4 *)state)[i] = make_int4(0, 0, 0, 0);
}

// Zeroes `n` launches' work queues (they must be zero when their kernel starts), for launches whose queues no launch before them has cleared.
static __global__ void queue_reset_kernel(WorkQueue *q, int n, int stride)
{
    int4 *w = (int4 *)q;
    for (int i = threadIdx.x; i < 8 * n; i += blockDim.x) w[i * stride] = make_int4(0, 0, 0, 0);
}

// Workgroups of `kernel` that the whole chip holds at once.
template <typename K>
static int resident_workgroups(K kernel, int threads)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess ||
        cus < 1 || per_cu < 1) {
        (void)hipGetLastError();
        return 0;  // unknown: the caller falls back to one workgroup per work item
    }
    return cus * per_cu;
}

// Workgroups of a kernel (a template argument) that the chip holds at once; queried once.
template <auto Kernel>
static int resident_of(int threads)
{
    static const int resident = resident_workgroups(Kernel, threads);
    return resident;
}

// A launch needs its queue only when there are more work items than the chip holds workgroups at
// once; otherwise one workgroup per item, all resident together, is the whole schedule.
template <auto Kernel>
static bool wants_queue(int threads, int n_work)
{
    const int resident = resident_of<Kernel>(threads);
    return resident > 0 && n_work > resident;
}

// Persistent launch when `queued` (as many workgroups as fit the chip at once, each taking work
// items until none is left), else a plain grid of one workgroup per item (`prm` then carries no queue).
template <auto Kernel>
static int launch_size(int threads, int n_work, bool queued) { return queued ? resident_of<Kernel>(threads) : n_work; }
