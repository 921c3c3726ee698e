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
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

struct WorkQueue {
    int32_t next[8];  // per die: how many of its work items have been handed out (but the first ones)
    int32_t pad[8];
};

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

// The work item that count `k` of die `xcd`'s queue stands for (a queue starts behind the items that
// the launch's workgroups took by their block index), or kQueueEmpty.
constexpr int kNoWork = -1, kQueueEmpty = -2;
__device__ __forceinline__ int queued_work(int n_work, int n_first, int xcd, int k)
{
    const int w = 8 * (k + (n_first - xcd + 7) / 8) + xcd;
    return w < n_work ? w : kQueueEmpty;
}

// The next item of the queue with the most items left; kNoWork when every queue is empty.  Called by
// one lane.  Counters are device-scope atomics (the dies' L2 caches are not coherent with
// each other for plain accesses).
__device__ __forceinline__ int stolen_work(WorkQueue *q, int n_work, int n_first)
{
    for (;;) {
        int best = -1, best_left = 0;
        for (int y = 0; y < 8; ++y) {
            const int ky = __hip_atomic_load(&q->next[y], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // items of queue y: ceil((n_work - y) / 8), without the first ones
            const int left = (n_work - y + 7) / 8 - (n_first - y + 7) / 8 - ky;
            if (left > best_left) { best_left = left; best = y; }
        }
        if (best < 0) return kNoWork;
        const int k = __hip_atomic_fetch_add(&q->next[best], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int w = queued_work(n_work, n_first, best, k);
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
// With `by_index` the first item is the one of the block index.  Blocks go to the compute units of a
// die in turn, so the workgroups that share a unit start with items a third or half of the first
// round apart; with items claimed in order of arrival a unit could start with three of the longest
// (30,934 tokens in 3 sequences, 4/4 heads of 64: forward 0.64 ms claimed, 0.48 by index).  Where a
// unit holds one workgroup and the items are alike, the order of arrival staggers them a little, and
// they run faster than in step (dK/dV, 27 sequences, 20,011 tokens, 32/8 heads of 128: 3 %).
// `slot` is one int of LDS; the caller has a barrier between a `take` and the next `post`.
struct WorkFeed {
    WorkQueue *q;
    int n_work, n_first, pending;  // items; how many are taken by block index (the workgroups of the launch, or none)
    int *slot;

    __device__ __forceinline__ int first()
    {
        if (n_first > 0 || !q) return (int)blockIdx.x;
        return again();
    }
    __device__ __forceinline__ void ask()
    {
        if (q && threadIdx.x == 0) {
            // (an address the compiler cannot see to be uniform: for a uniform one it adds up the
            // lanes that are on, one here, and waits for the answer at once to spread it to them)
            uint32_t die;
            int one;
            asm volatile("v_mov_b32 %0, %2\n\tv_mov_b32 %1, 1" : "=v"(die), "=v"(one) : "s"(my_xcd()));
            pending = __hip_atomic_fetch_add(&q->next[die], one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __device__ __forceinline__ void post()
    {
        if (q && threadIdx.x == 0) *slot = queued_work(n_work, n_first, my_xcd(), pending);
    }
    __device__ __forceinline__ int take() const { return q ? __builtin_amdgcn_readfirstlane(*slot) : kNoWork; }
    // after kQueueEmpty: an item of another die's queue
    __device__ __forceinline__ int other()
    {
        __syncthreads();  // everyone has read the slot
        if (threadIdx.x == 0) *slot = stolen_work(q, n_work, n_first);
        __syncthreads();
        return take();
    }
    // all of it at once, for a workgroup that has no work to hide it behind
    __device__ __forceinline__ int again()
    {
        if (!q) return kNoWork;
        __syncthreads();  // everyone has read the slot
        ask();
        post();
        __syncthreads();
        const int w = take();
        return w == kQueueEmpty ? other() : w;
    }
};

// Zeroes `n` work queues (a launch's queue must be zero when its kernel starts).
static __global__ void queue_reset_kernel(WorkQueue *q, int n)
{
    int32_t *w = (int32_t *)q;
    for (int i = threadIdx.x; i < n * (int)(sizeof(WorkQueue) / 4); i += blockDim.x) w[i] = 0;
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
