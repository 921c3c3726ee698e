// Varlen descriptor builder and cost-ordered tile work lists, on the device.
//
// The micro-batch is stated the way the paper states it (Sec. 4.1, Eq. 1-8):
// full lengths S[K] plus, per sequence, local (degree 1) or distributed over N
// ranks with this GPU holding slice `index` (Eq. 8: S_k/N tokens per rank), cut
// either as one contiguous slice or as two chunks that balance the causal work.
// Four small kernels, or, for a small micro-batch, one workgroup that does what they do (plan_small):
//   1. plan_ranges : per-segment query/KV ranges, the packed offsets
//                    (exclusive scans), per-segment work-item offsets, totals
//   2. plan_emit   : one thread per work item writes {seq, block, x, cost}
//   3. plan_sort   : stable descending-cost order by rank counting, so the
//                    hardware dispatcher, which hands out workgroups in grid
//                    order, always gives the heaviest remaining tile to the
//                    first compute unit that frees up -- the paper's
//                    least-loaded-first rule (Alg. 1, argmin over L) applied
//                    to compute units instead of ranks.
//   4. plan_units  : which dK/dV items several workgroups share, and the lists of work units
#include "common.h"

namespace {

constexpr int kScanThreads = 256;

// Block-wide exclusive scan of one int64 per thread; returns the exclusive
// prefix and writes the block total to *total (same value in every thread).
// Inside a wavefront the scan runs on lane shuffles; the four wavefronts' totals
// meet in LDS (two barriers per scan).
__device__ inline int64_t block_exclusive_scan(int64_t v, int64_t *lds, int64_t *total)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int64_t incl = v;
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t up = __shfl_up(incl, off, 64);
        if (lane >= off) incl += up;
    }
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    int64_t before = 0, all = 0;
    for (int w = 0; w < kScanThreads / 64; ++w) {
        const int64_t x = lds[w];
        if (w < wave) before += x;
        all += x;
    }
    *total = all;
    __syncthreads();  // lds may be reused by the next scan
    return before + incl - v;
}

// Block-wide maximum of one non-negative int64 per thread, in every thread.
__device__ inline int64_t block_max(int64_t v, int64_t *lds)
{
    for (int off = 32; off > 0; off >>= 1) {
        const int64_t o = __shfl_xor(v, off, 64);
        v = o > v ? o : v;
    }
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    for (int w = 0; w < kScanThreads / 64; ++w) v = lds[w] > v ? lds[w] : v;
    __syncthreads();  // lds may be reused
    return v;
}

__device__ inline int64_t wave_sum(int64_t v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
__device__ inline int32_t wave_max(int32_t v)
{
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
    return v;
}

__device__ inline int64_t ceil_div64(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Choice between BN and a larger dK/dV block bn_alt (0 = no choice to make).  The larger
// one is taken when, with blocks of BN key rows, the costliest work item exceeds an even
// share of the whole list over the compute units (cost_max > cost_sum * Hkv / CUs), the
// same ratio that decides the head split; the costs are those of the dK/dV items that
// plan_emit_kernel would write for BN.  It is also taken, given a sequence of at least two
// of the larger blocks, when their list is still long (at least five x KV heads per compute
// unit) or when the costliest item stays under 0.7 of that even share.  Fewer, larger
// workgroups run the rounds 7-18 % faster (measured on 14 to 64 heads x 16,384-65,536 tokens,
// uniform and ragged lengths) but balance worse: with few items and a costliest one between
// 0.7 and 1.0 of the even share, ragged micro-batches lost 4-15 % by them.
__device__ inline bool larger_key_blocks(int64_t c_sum, int64_t c_max, int64_t n_alt, int64_t longest, int32_t bn_alt, int32_t kv_heads,
                                         int32_t compute_units)
{
    const bool long_list = n_alt * kv_heads >= 5 * (int64_t)compute_units;
    const bool even_list = 10 * c_max * compute_units <= 7 * c_sum * kv_heads;
    return c_max * compute_units > c_sum * kv_heads || ((long_list || even_list) && longest >= 2 * (int64_t)bn_alt);
}

// One thread per sequence.  A sequence cut the contiguous way is one query
// segment; one cut the load-balanced way (chunks r and 2N-1-r of 2N) is two
// consecutive segments, early chunk first, that share one key/value prefix (the
// late chunk's).  All per-segment arrays are indexed by segment; fwd_off / dkv_off
// are the work-item offsets (an early chunk owns no dK/dV items: its offset equals
// its partner's).
__global__ __launch_bounds__(kScanThreads) void plan_ranges_kernel(
    const int32_t *__restrict__ S, const int32_t *__restrict__ N, const int32_t *__restrict__ R,
    const int32_t *__restrict__ Z, int32_t K, int32_t BM, int32_t BN, int32_t max_q_rows,
    int32_t max_k_rows, int32_t *__restrict__ q_begin, int32_t *__restrict__ q_len,
    int32_t *__restrict__ kv_len, int32_t *__restrict__ cu_q, int32_t *__restrict__ cu_k,
    int32_t *__restrict__ shares_kv, int32_t *__restrict__ fwd_off, int32_t *__restrict__ dkv_off,
    int32_t cap_fwd, int32_t cap_dkv, int32_t bn_alt, int32_t kv_heads, int32_t compute_units,
    PlanTotals *__restrict__ totals)
{
    __shared__ int64_t lds[kScanThreads];
    __shared__ int32_t first_bad;
    const int t = threadIdx.x;
    if (t == 0) first_bad = 0x7fffffff;
    __syncthreads();
    if (bn_alt != 0) {
        // (BM is a power of two and positions fit 32 bits: divided in 64 bits, this walk over the blocks
        // of one 3,629-token sequence was most of the 16 us that the kernel took; now 11)
        int64_t c_sum = 0, c_max = 0, n_alt = 0, longest = 0;
        const int log_bm = __ffs(BM) - 1;
        for (int32_t k = t; k < K; k += kScanThreads) {
            const int64_t s = S[k], n = N[k], r = R[k], z = Z[k];
            const int64_t chunks = n * (z ? 2 : 1);
            if (s < 1 || n < 1 || r < 0 || r >= n || (z != 0 && z != 1) || chunks > s) continue;
            const int64_t idx[2] = {r, 2 * n - 1 - r};
            const int nseg = (int)z + 1;
            int32_t qb[2] = {0, 0}, qe[2] = {0, 0};
            for (int part = 0; part < nseg; ++part) {
                qb[part] = chunks == 1 ? 0 : (int32_t)((idx[part] * s) / chunks);
                qe[part] = chunks == 1 ? (int32_t)s : (int32_t)(((idx[part] + 1) * s) / chunks);
            }
            const int32_t end = qe[nseg - 1];
            n_alt += (uint32_t)(end + bn_alt - 1) / (uint32_t)bn_alt;
            longest = end > longest ? end : longest;
            for (int64_t j0 = 0; j0 < end; j0 += BN) {
                int32_t cost = 0;
                for (int part = 0; part < nseg; ++part) {
                    if (j0 >= qe[part]) continue;
                    const int32_t i0 = j0 > qb[part] ? (int32_t)j0 - qb[part] : 0;
                    cost += ((qe[part] - qb[part] - 1) >> log_bm) + 1 - (i0 >> log_bm);
                }
                c_sum += cost;
                c_max = cost > c_max ? cost : c_max;
            }
        }
        int64_t tot;
        block_exclusive_scan(c_sum, lds, &tot);
        c_sum = tot;
        c_max = block_max(c_max, lds);
        block_exclusive_scan(n_alt, lds, &tot);
        n_alt = tot;
        longest = block_max(longest, lds);
        if (larger_key_blocks(c_sum, c_max, n_alt, longest, bn_alt, kv_heads, compute_units))
            BN = bn_alt;
    }
    int64_t base_s = 0, base_q = 0, base_k = 0, base_f = 0, base_d = 0, pairs = 0;
    for (int32_t k0 = 0; k0 < K; k0 += kScanThreads) {
        const int32_t k = k0 + t;
        int64_t qb[2] = {0, 0}, ql[2] = {0, 0}, nf[2] = {0, 0};
        int64_t nseg = 0, owned = 0, nd = 0, pr = 0;
        if (k < K) {
            const int64_t s = S[k], n = N[k], r = R[k], z = Z[k];
            const int64_t chunks = n * (z ? 2 : 1);
            if (s < 1 || n < 1 || r < 0 || r >= n || (z != 0 && z != 1) || chunks > s) {
                atomicMin(&first_bad, k);
            } else {
                nseg = z + 1;
                const int64_t idx[2] = {r, 2 * n - 1 - r};
                for (int part = 0; part < nseg; ++part) {
                    const int64_t b = (idx[part] * s) / chunks, e = ((idx[part] + 1) * s) / chunks;
                    qb[part] = b;
                    ql[part] = e - b;
                    nf[part] = ceil_div64(e - b, BM);
                    pr += (e * (e + 1) - b * (b + 1)) / 2;
                    owned = e;  // the late chunk's prefix covers the early one's
                }
                // one sequence of one tensor must span fewer than 2^31 elements
                // (the kernels address inside a sequence with 32-bit offsets)
                if (ql[0] + ql[1] > max_q_rows || owned > max_k_rows) atomicMin(&first_bad, k);
                nd = ceil_div64(owned, BN);
            }
        }
        int64_t tot;
        const int64_t e_s = block_exclusive_scan(nseg, lds, &tot);
        const int64_t seg0 = base_s + e_s;
        base_s += tot;
        const int64_t e_q = block_exclusive_scan(ql[0] + ql[1], lds, &tot);
        const int64_t row0 = base_q + e_q;
        base_q += tot;
        const int64_t e_k = block_exclusive_scan(owned, lds, &tot);
        const int64_t krow0 = base_k + e_k;
        base_k += tot;
        const int64_t e_f = block_exclusive_scan(nf[0] + nf[1], lds, &tot);
        const int64_t f0 = base_f + e_f;
        base_f += tot;
        const int64_t e_d = block_exclusive_scan(nd, lds, &tot);
        const int64_t d0 = base_d + e_d;
        base_d += tot;
        block_exclusive_scan(pr, lds, &tot);
        pairs += tot;
        for (int part = 0; part < nseg; ++part) {
            const int64_t sg = seg0 + part;
            q_begin[sg] = (int32_t)qb[part];
            q_len[sg] = (int32_t)ql[part];
            kv_len[sg] = (int32_t)(qb[part] + ql[part]);
            cu_q[sg] = (int32_t)(row0 + (part ? ql[0] : 0));
            cu_k[sg] = (int32_t)krow0;
            shares_kv[sg] = part;
            fwd_off[sg] = (int32_t)(f0 + (part ? nf[0] : 0));
            dkv_off[sg] = (int32_t)d0;
        }
    }
    __syncthreads();
    if (t == 0) {
        cu_q[base_s] = (int32_t)base_q;
        cu_k[base_s] = (int32_t)base_k;
        fwd_off[base_s] = (int32_t)base_f;
        dkv_off[base_s] = (int32_t)base_d;
        totals->total_q = base_q;
        totals->total_k = base_k;
        totals->n_fwd = base_f;
        totals->n_dkv = base_d;
        totals->pairs = pairs;
        totals->bad_entry = (first_bad == 0x7fffffff) ? 0 : first_bad + 1;
        totals->n_seg = (int32_t)base_s;
        totals->dkv_cost_sum = 0;
        totals->dkv_cost_max = 0;
        for (int i = 0; i <= SKRULL_CHAIN_LIMITS; ++i) totals->chain_hist[i] = 0;
        for (int i = 0; i < SKRULL_UNIT_LISTS; ++i) totals->n_units[i] = 0;
        totals->n_dkv_units = totals->fwd_longest = totals->fwd_longest_full = 0;
        totals->fwd_load = 0;
        totals->cap_fwd = cap_fwd;
        totals->cap_dkv = cap_dkv;
        totals->block_n = BN;
    }
}

// Offsets of up to this many segments are searched in LDS: a search in memory is a chain of
// log2(K) loads, half of the emit kernel's time for a few dozen sequences.
constexpr int32_t kEmitSegments = 1024;

// Largest k with off[k] <= item (off is an exclusive scan with off[K] = n).
__device__ inline int32_t owner_of(const int32_t *off, int32_t K, int32_t item)
{
    int32_t lo = 0, hi = K;  // invariant: off[lo] <= item < off[hi]
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (off[mid] <= item) lo = mid; else hi = mid;
    }
    return lo;
}

// The plan's queues start empty (by all threads of one workgroup).
__device__ inline void clear_sets(int4 *sets)
{
    static_assert(SKRULL_SETS_INTS % 4 == 0, "cleared in fours");
    for (int i = threadIdx.x; i < SKRULL_SETS_INTS / 4; i += blockDim.x) sets[i] = make_int4(0, 0, 0, 0);
}

__global__ __launch_bounds__(256) void plan_emit_kernel(
    int32_t K, int32_t BM, const int32_t *__restrict__ q_begin,
    const int32_t *__restrict__ q_len, const int32_t *__restrict__ kv_len,
    const int32_t *__restrict__ cu_q, const int32_t *__restrict__ shares_kv,
    const int32_t *__restrict__ fwd_off,
    const int32_t *__restrict__ dkv_off, int4 *__restrict__ fwd_items,
    int4 *__restrict__ dkv_items, PlanTotals *__restrict__ totals, int4 *__restrict__ sets)
{
    if (blockIdx.x == 0) clear_sets(sets);
    // the grid covers an upper bound of the item counts; the counts themselves are the
    // ranges kernel's (clamped: a count past the limit is rejected by the host afterwards)
    const int32_t n_fwd = (int32_t)min((long long)totals->n_fwd, (long long)totals->cap_fwd);
    const int32_t n_dkv = (int32_t)min((long long)totals->n_dkv, (long long)totals->cap_dkv);
    const int32_t BN = totals->block_n;  // the ranges kernel's choice where the caller left it open
    const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    __shared__ int32_t off_f[kEmitSegments + 1], off_d[kEmitSegments + 1];
    if (K <= kEmitSegments) {
        for (int32_t i = threadIdx.x; i <= K; i += blockDim.x) {
            off_f[i] = fwd_off[i];
            off_d[i] = dkv_off[i];
        }
        __syncthreads();
    }
    if (t < n_fwd) {
        const int32_t k = K <= kEmitSegments ? owner_of(off_f, K, t) : owner_of(fwd_off, K, t);
        const int32_t m = t - fwd_off[k];
        const int64_t row0 = (int64_t)m * BM;
        const int64_t left = q_len[k] - row0;
        const int64_t rows = left < BM ? left : BM;
        fwd_items[t] = make_int4(k, m, (int32_t)(cu_q[k] + row0),
                                 (int32_t)((uint32_t)(q_begin[k] + row0 + rows + BN - 1) / (uint32_t)BN));  // (below 2^31 + 256)
    }
    if (t < n_dkv) {
        // equal offsets (an early chunk and its partner) resolve to the later segment,
        // the one that owns the shared prefix
        const int32_t k = K <= kEmitSegments ? owner_of(off_d, K, t) : owner_of(dkv_off, K, t);
        const int32_t b = t - dkv_off[k];
        int64_t i0 = (int64_t)b * BN - q_begin[k];
        if (i0 < 0) i0 = 0;
        const int log_bm = __ffs(BM) - 1;  // a power of two
        const int32_t m0 = (int32_t)(i0 >> log_bm);
        int32_t cost = ((q_len[k] - 1) >> log_bm) + 1 - m0;
        if (shares_kv[k] && (int64_t)b * BN < kv_len[k - 1]) {  // query blocks of the early chunk
            int64_t j0 = (int64_t)b * BN - q_begin[k - 1];
            if (j0 < 0) j0 = 0;
            cost += ((q_len[k - 1] - 1) >> log_bm) + 1 - (int32_t)(j0 >> log_bm);
        }
        dkv_items[t] = make_int4(k, b, m0, cost);
        atomicAdd(&totals->dkv_cost_sum, (unsigned long long)cost);
        atomicMax(&totals->dkv_cost_max, cost);
    }
}

// Counts a dK/dV item of cost `cost` by the length of its chain of `group` heads.  The base of the
// limits balances two losses: workgroups that share an item each pay its start, its end and its
// partial sums (as much as one to two blocks' rounds), so short parts are dear, and units that are
// long against an even share s of the whole list per compute unit balance badly.  The first loss
// falls and the second grows with the length: sqrt(8 s), at least 2 blocks and, at head_dim 64, at
// most 13.  On 82 micro-batches a quarter, half, twice and four times that change dK/dV on 22, by
// +9, +4, +1 and +28 % on (geometric) average (profiles/chain_limit_sweep.txt).
// A workgroup counts in LDS and adds its ten counts to the totals once: item by item into the totals, the atomics on
// these few words were most of the sort (950 and 1,719 items: 39 us, 16 this way; the call 115 and 92).
struct ChainCounts {
    int32_t base, hist[SKRULL_CHAIN_LIMITS + 1];  // of a workgroup, in LDS
    // by all threads; a barrier has to follow
    __device__ void begin(const PlanTotals *totals, int32_t q_heads, int32_t head_dim, int32_t compute_units)
    {
        if (threadIdx.x <= SKRULL_CHAIN_LIMITS) hist[threadIdx.x] = 0;
        const float share = (float)totals->dkv_cost_sum * (float)q_heads / (float)compute_units;
        const float best = fminf(sqrtf(8.0f * share), head_dim == 64 ? 13.0f : 1e6f);
        if (threadIdx.x == 0) base = max(2, (int32_t)best);
    }
    __device__ void count(int32_t cost, int32_t group)
    {
        const int64_t chain = (int64_t)cost * group;
        int above = 0;
        while (above < SKRULL_CHAIN_LIMITS && chain > dkv_chain_limit(base, above)) ++above;
        atomicAdd(&hist[above], 1);
    }
    // by all threads, after a barrier
    __device__ void end(PlanTotals *totals)
    {
        if (threadIdx.x <= SKRULL_CHAIN_LIMITS && hist[threadIdx.x] > 0) atomicAdd(&totals->chain_hist[threadIdx.x], hist[threadIdx.x]);
        if (threadIdx.x == 0) totals->chain_base = base;  // (the same from every workgroup)
    }
};

// Stable sort by descending .w: item a goes to slot
//   #{b : cost_b > cost_a} + #{b < a : cost_b == cost_a}.
// Costs are streamed through LDS in tiles; four threads walk a tile for one item, four costs to a
// read.  (One thread per item and one cost to a read, each waited for, took 12 us for 180 items and
// 25 us for 310; both lists together now take 14 for 1,054 and 1,318.)  blockIdx.y: the list (0 forward / dQ, 1 dK/dV).
constexpr int32_t kSortItems = 64;  // items of a block
struct SortJob {
    const int4 *in;
    int4 *out;
};
__global__ __launch_bounds__(256) void plan_sort_kernel(SortJob fwd, SortJob dkv, int first_list, PlanTotals *totals,
                                                        int32_t group, int32_t q_heads, int32_t head_dim,
                                                        int32_t compute_units)
{
    __shared__ __align__(16) int32_t tile[1024];
    __shared__ ChainCounts chains;
    const int which = first_list + blockIdx.y;
    const int4 *__restrict__ in = which == 0 ? fwd.in : dkv.in;
    int4 *__restrict__ out = which == 0 ? fwd.out : dkv.out;
    const int32_t n = which == 0 ? (int32_t)min((long long)totals->n_fwd, (long long)totals->cap_fwd)
                                 : (int32_t)min((long long)totals->n_dkv, (long long)totals->cap_dkv);
    const int32_t first = blockIdx.x * kSortItems;
    if (first >= n) return;  // (the whole block)
    if (which == 1) chains.begin(totals, q_heads, head_dim, compute_units);  // (barriers follow: n > 0)
    const int32_t a = first + threadIdx.x / 4, quarter = threadIdx.x % 4;
    const int4 me = (a < n) ? in[a] : make_int4(0, 0, 0, 0);
    int32_t rank = 0;
    for (int32_t b0 = 0; b0 < n; b0 += 1024) {
        __syncthreads();
        const int32_t lim = (n - b0 < 1024) ? n - b0 : 1024;
        for (int32_t i = threadIdx.x; i < ((lim + 15) & ~15); i += blockDim.x) {
            tile[i] = i < lim ? in[b0 + i].w : -1;  // (below every cost)
        }
        __syncthreads();
        // cost_b > cost_a, or equal and earlier: cost_b >= cost_a + (b >= a)
        const int32_t before = a - b0;
        for (int32_t x = 4 * quarter; x < lim; x += 16) {
            const int4 c = *(const int4 *)&tile[x];
            rank += (c.x >= me.w + (x >= before)) + (c.y >= me.w + (x + 1 >= before)) +
                    (c.z >= me.w + (x + 2 >= before)) + (c.w >= me.w + (x + 3 >= before));
        }
    }
    rank += __shfl_xor(rank, 1, 64);
    rank += __shfl_xor(rank, 2, 64);
    if (a < n && quarter == 0) {
        out[rank] = me;
        if (which == 1) chains.count(me.w, group);
    }
    if (which != 1) return;
    __syncthreads();
    chains.end(totals);
}

// ---------------------------------------------------------------------------
// How dK/dV items are shared, and in which order work is handed out.
// ---------------------------------------------------------------------------

// dK/dV head split.  A workgroup of that kernel walks all query tiles of one key
// block for every query head of the KV group, one after another; its longest chain
// is cost_max * group.  Spread evenly, the whole list is cost_sum * group * Hkv over
// the compute units.  When the longest chain exceeds that share (few KV heads, one
// long sequence in a small micro-batch) the heads of a group are shared out over
// several workgroups until it no longer does, with a factor two of slack.
//
// Split only when the longest chain of the work list (its costliest item, all the
// heads of a group) exceeds an even share of the whole list over the compute units:
// then that chain bounds the kernel's time and shortening it pays for the fp32
// partial sums and their reduction; below that the unsplit kernel is 5-40 % faster
// (measured on 45 micro-batches of three head shapes; the ratio below was the
// dividing line at 1.0: splits won from 1.27 up, lost or tied up to 0.98).
// The 12-wavefront shape (fewer, larger workgroups: rounding of workgroups per compute
// unit weighs more) gains from the split from half that ratio on: at 14/2 heads x 64
// every batch measured from 2 x 8,192 to 65,536 tokens was 7-50 % faster split 7 ways
// (65,536 tokens, ratio 0.75: 17.4 -> 16.1 ms; eight 8,192-token sequences, 0.72: equal).
__device__ inline int32_t choose_head_split(const PlanTotals &totals, int32_t q_heads, int32_t kv_heads, int32_t head_dim,
                                            int32_t longest_seq, int32_t compute_units)
{
    const int32_t group = q_heads / kv_heads;
    const double share = (double)totals.dkv_cost_sum * kv_heads / (double)compute_units;
    // (that factor of two only where it was measured to pay: a sequence of 8,192 tokens or more
    // and a short list, under five items x KV heads per compute unit; with longer lists of
    // 192-key items, 16-64 heads on ragged 32,768-token micro-batches, a split at ratios of
    // 0.6-0.9 cost 6-16 %, and on short lists of short sequences up to 90 %)
    const bool short_list = (int64_t)totals.n_dkv * kv_heads < 5 * (int64_t)compute_units;
    const double scale = (head_dim == 64 && totals.block_n == 192 && short_list && longest_seq >= 8192) ? 2.0 : 1.0;
    const double want = share > 0.0 ? scale * (double)totals.dkv_cost_max / share : 1.0;
    int32_t hs = want <= 1.0 ? 1 : (want >= (double)group ? group : (int32_t)ceil(want));
    // only equal shares: workgroups with different numbers of heads walk the query
    // tiles at different paces, stop sharing them in L2 and run 10 % slower (measured
    // with 7 heads per group split 3 + 4), so take the next divisor of the group size
    const int32_t wanted = hs;
    while (hs < group && group % hs != 0) ++hs;
    // ... unless that divisor is three times what was asked for and the chain is less than
    // 1.5 even shares (7 heads per group at ratios of 1.0-1.4: split 7 ways 6-14 % slower
    // than unsplit, equal at 1.7)
    if (hs >= 3 * wanted && want < 1.5) hs = 1;
    return hs < 1 ? 1 : (hs > group ? group : hs);
}

// Which dK/dV items are shared out over several workgroups.  A head split the caller asked for holds
// for every item.  The library's own shares out only items with a long chain: split over the heads,
// every item of a short sequence cost seven starts, seven ends and seven fp32 partial sums instead of
// one store (64 sequences, 26,624 tokens, 14/2 heads of 64: dK/dV 202 us all items split 7 ways,
// 146 this way; 20 sequences, 16,384 tokens: 184 -> 162), and where the heads cannot be split evenly
// the longest chain was the kernel's time (10 sequences, 13,312 tokens, 28/4 heads of 128: 640 -> 530;
// one of 2,967, 4/4 heads of 64: 69 -> 36).
__device__ inline SplitChoice choose_split(int32_t asked, const PlanTotals &totals, int32_t q_heads, int32_t kv_heads, int32_t head_dim,
                                           int32_t longest_seq, int32_t compute_units)
{
    const int32_t group = q_heads / kv_heads;
    SplitChoice r{asked, 0, 0, 1, 0, 0};
    if (asked != 0) {
        if (asked > 1) {
            r.parts = asked;
            r.n_split = (int32_t)totals.n_dkv;
        }
        return r;
    }
    r.head_split = choose_head_split(totals, q_heads, kv_heads, head_dim, longest_seq, compute_units);
    const int64_t longest = (int64_t)totals.dkv_cost_max * group;
    // Where the heads are not split (nor could be: one head per group, or seven, which would be too many)
    // items are shared out only if the longest chain exceeds 1.1 even shares, if its shortening saves more
    // than the partial sums cost, and as few as it takes for these to fit the static workspace, so that a
    // plan that skrull_attn_bwd_static takes without them is not refused for them.
    r.compact = r.head_split == 1;
    if (r.compact && 10 * longest * compute_units <= 11 * (int64_t)totals.dkv_cost_sum * q_heads) return r;
    // Microseconds: a block of 256 query rows of one head takes a workgroup 6, the partial sums are written
    // and read at 4.4 TB/s, and a part's start and end take 6, or 1 where compute units are idle beside it.
    // Measured on 170 micro-batches of ratios from 1.1 up, shared against whole: where this says no, up to 27 %
    // slower (a slice of 2,388 tokens, 4/4 heads of 64, ratio 1.43 and 33 MB: 86 us shared, 68 whole); where
    // it says yes, 3 % slower (a microsecond of 40) to 50 % faster (28/4 heads of 128, ratio 1.14 and 17 MB:
    // 662 us shared, 816 whole; one sequence of 2,967, 4/4 heads of 64, ratio 7 and 19 MB: 34 and 69).
    auto pays = [&](int64_t limit) {
        const double share = (double)totals.dkv_cost_sum * q_heads / compute_units;
        const double saved = (double)longest - (share > (double)limit ? share : (double)limit);
        return 6.0 * saved > ((double)longest < 2.0 * share ? 6.0 : 1.0) + 2.0 * (double)partial_bytes(r, totals.block_n, totals.total_k, kv_heads, head_dim) / 4.4e6;
    };
    const int32_t most = r.compact ? kMaxParts : r.head_split;
    // When the longest part is then still as long as three quarters of an even share, all items are cut
    // as fine as it is: what else runs has to fit beside it (3 sequences, 7,417 tokens, 14/2 heads of
    // 64: dK/dV 137 us all cut, 145 by the limits below).
    if (!r.compact && 4 * longest * compute_units >= 3 * most * (int64_t)totals.dkv_cost_sum * q_heads) {
        r.parts = most;
        r.n_split = (int32_t)totals.n_dkv;
        return r;
    }
    int32_t above[SKRULL_CHAIN_LIMITS + 1];  // items that exceed limit k
    above[SKRULL_CHAIN_LIMITS] = 0;
    for (int k = SKRULL_CHAIN_LIMITS - 1; k >= 0; --k) above[k] = above[k + 1] + totals.chain_hist[k + 1];
    for (int k = 2; k < SKRULL_CHAIN_LIMITS; ++k) {
        const int64_t limit = dkv_chain_limit(totals.chain_base, k), want = (longest + limit - 1) / limit;
        if (want < 2) break;
        r.parts = want > most ? most : (int32_t)want;
        r.chain = (int32_t)(limit > INT32_MAX ? INT32_MAX : limit);
        r.n_split = above[k];
        r.n_whole_first = above[k - 2] - above[k];
        if (!r.compact ||
            (pays(limit) && base_workspace(q_heads, totals.total_q) + partial_bytes(r, totals.block_n, totals.total_k, kv_heads, head_dim) <= (int64_t)SKRULL_STATIC_SCRATCH_BYTES)) return r;
    }
    r.parts = 1;
    r.n_split = r.n_whole_first = 0;
    return r;
}

// A dK/dV item of cost `cost` among the first n_split is shared by this many workgroups.
__device__ inline int32_t parts_of_item(const SplitChoice &c, int32_t item, int32_t cost, int32_t group)
{
    if (item >= c.n_split) return 1;
    return c.chain == 0 ? c.parts : (int32_t)min((int64_t)c.parts, ((int64_t)cost * group + c.chain - 1) / c.chain);
}

// The order in which work is handed out: the longest first, as in the item lists, but by what a work
// unit takes: for dK/dV an item's part by its rounds (64-row query tiles x heads), for the forward and dQ
// at head_dim 64 an item by its half tiles of keys.  The items' own costs count blocks of 256 rows, in which most short
// sequences look alike, and whole items went out before the parts of shared ones, whatever their
// length: launches ended with long units that had begun late.  dQ and dK/dV together, by the items' costs
// and this way: 64 sequences, 26,624 tokens, 14/2 heads of 64: 240 -> 229 us; 20 sequences, 16,384 tokens: 248 ->
// 236; 114 sequences of 16 to 1,024, 32,768 tokens: 218 -> 198; 10 sequences, 13,312 tokens, 28/4 heads of 128: 857
// -> 845.  The forward gains 1 % at head_dim 64 (at 128 neither it nor dQ gains).
// What is not done, because units that read the same tiles find them in their die's L2 when they run together:
//  the parts of a forward / dQ item apart from each other by their own half tiles (114 sequences of about 250
//    tokens, 32/8 heads of 128: forward 215 -> 236, dQ 303 -> 328);
//  the key blocks of a short sequence apart from each other: they go out by the sequence's length, the rounds of its
//    first block, where these are at most `small` (114 sequences of about 250 tokens, 32/8 heads of 128: dK/dV 359 us,
//    by their own rounds 368, by the items' costs 371; 26,624 tokens above 134, 137, 146).  `small` is an eighth of an
//    even share per compute unit, or a quarter at head_dim 128 where no item is shared, and 64 at most (128 is the same): these blocks
//    are what fills the end of a launch, and 1,187 rounds, a quarter of the share of 24,576 + 8,192 tokens at
//    32/8 heads of 128, brought them out before it (8,660 us, 8,540 this way, 8,522 by the items' costs).  Where the KV
//    heads are a multiple of the eight dies, neighbours in the list with the same head are on the same die, and `small` is half
//    a share if no block takes longer than that, or than 24 rounds (8/8 heads of 128: 32 sequences of 256 34 us, 38 by their own rounds; 33 of 511
//    71 and 79; 16/16 heads of 64: 16 of 512 46 and 48).  With half a share elsewhere launches end worse: neighbours are on
//    different dies (28/4 heads of 128: 63 of 130 68 us, 92 that way; 14/2 heads of 64: 128 of 256 75 and 88), or the short
//    blocks are what is left to fill the end (5,866 and 1,546 tokens, 16/16 heads of 64: 175 and 190; a cut of 18,174 over 8
//    ranks beside 1,024 and 463 201 and 210);
//  at head_dim 128 with KV heads a multiple of the dies and no shared items, neighbouring key blocks of one length in blocks of
//    256 rows apart from each other, where a launch has 3.5 workgroups and more per compute unit: those go out by the
//    items' costs, and short sequences together up to 32 rounds.  (Of 252 micro-batches of six such head shapes 204 have so many: against the items'
//    costs with nothing kept together their own rounds take from 7 % less to 7 % more time, this way from 7 % less to 2 % more; 2,500 and 30 of
//    700 tokens, 32/8 heads: 410, 439, 402 us; 32 of 1,024, 64/8 heads: 1,203, 1,255, 1,192.  The other 48 take 4 % less on average by their
//    own rounds; 16 of 512, 32/8 heads: 101 us by the items' costs, 91 by those);
//  any order but the list's where all units run at once (4,923 tokens, 28/4 heads of 128: 111 us, else 114).
struct UnitCosts {
    const int32_t *q_begin, *q_len, *kv_len, *shares_kv;
    int32_t BM, BN, group, head_dim;
    SplitChoice choice;
    int32_t small;
    bool by_items;
    // query tiles of a segment that see key kv0 or later ones
    __device__ int32_t tiles(int32_t seq, int32_t kv0) const
    {
        const int32_t i0 = max(0, kv0 - q_begin[seq]);
        return ((q_len[seq] + 63) >> 6) - (i0 >> 6);
    }
    // item `i` of the sorted dK/dV list: what a part of it costs, and how many there are
    __device__ void dkv(const int4 &it, int32_t i, int32_t &cost, int32_t &parts) const
    {
        int32_t c = tiles(it.x, it.y * BN), whole = tiles(it.x, 0);
        if (shares_kv[it.x]) {
            whole += tiles(it.x - 1, 0);
            if (it.y * BN < kv_len[it.x - 1]) c += tiles(it.x - 1, it.y * BN);
        }
        parts = parts_of_item(choice, i, it.w, group);
        whole = min(whole, 1 << 20) * group;
        if (by_items) c = it.w * (BM >> 6);
        cost = whole <= small ? whole : (min(c, 1 << 20) * group + parts - 1) / parts;
    }
    // item of the forward / dQ list for workgroups of `waves` waves
    __device__ void fwd(const int4 &it, int32_t waves, int32_t &cost, int32_t &parts) const
    {
        const int32_t row0 = it.y * BM, rows = min(BM, q_len[it.x] - row0);
        cost = head_dim == 64 ? (int32_t)(((uint32_t)(q_begin[it.x] + row0 + rows) + 31u) >> 5) : 0;
        parts = (((rows + 31) >> 5) * group + waves - 1) / waves;
    }
    __device__ bool more_than_four_blocks(const int4 &it) const { return min(BM, q_len[it.x] - it.y * BM) > 128; }
};
__device__ inline bool by_item_costs(const PlanTotals &totals, const SplitChoice &choice, int32_t kv_heads, int32_t head_dim, int32_t compute_units)
{
    const int64_t workgroups = (int64_t)totals.n_dkv * ((totals.block_n + 127) / 128) * kv_heads;
    return head_dim == 128 && kv_heads % 8 == 0 && choice.parts == 1 && 2 * workgroups >= 7 * (int64_t)compute_units;
}
__device__ inline int32_t small_block(const PlanTotals &totals, const SplitChoice &choice, int32_t q_heads, int32_t kv_heads, int32_t head_dim,
                                      int32_t compute_units)
{
    // (a cost counts for four rounds)
    const unsigned long long half = 2 * totals.dkv_cost_sum * q_heads / (unsigned long long)compute_units;
    const bool all_short = kv_heads % 8 == 0 && 4ull * totals.dkv_cost_max * (q_heads / kv_heads) <= min(half, 24ull);
    if (all_short) return (int32_t)min(half, 64ull);
    return (int32_t)min(half / (head_dim == 64 || choice.parts > 1 ? 4 : 2), by_item_costs(totals, choice, kv_heads, head_dim, compute_units) ? 32ull : 64ull);
}
struct UnitsJob {
    const int4 *fwd_items, *dkv_items;
    const int32_t *q_begin, *q_len, *kv_len, *shares_kv;
    int32_t BM, q_heads, kv_heads, head_dim, asked, longest_seq, compute_units;
    int32_t *units[SKRULL_UNIT_LISTS];  // null: no list
    int4 *dkv_units;
};
__global__ __launch_bounds__(256) void plan_units_kernel(UnitsJob j, PlanTotals *totals)
{
    __shared__ __align__(16) int32_t t_cost[1024], t_parts[1024];
    __shared__ SplitChoice shared_choice;
    const int32_t group = j.q_heads / j.kv_heads;
    const int32_t first = blockIdx.x * kSortItems;
    const bool dkv = blockIdx.y == 0;
    if (dkv && threadIdx.x == 0) {
        const PlanTotals t = *totals;
        shared_choice = choose_split(j.asked, t, j.q_heads, j.kv_heads, j.head_dim, j.longest_seq, j.compute_units);
        if (blockIdx.x == 0) totals->split = shared_choice;  // (read by the host only)
    }
    const int32_t n = dkv ? (int32_t)min((long long)totals->n_dkv, (long long)totals->cap_dkv)
                          : (int32_t)min((long long)totals->n_fwd, (long long)totals->cap_fwd);
    const int32_t NW = 4 * blockIdx.y;  // forward / dQ: waves of a workgroup
    int32_t *units = dkv ? nullptr : j.units[blockIdx.y - 1];
    if ((dkv ? !j.dkv_units : !units) || first >= n) return;  // (the whole block)
    __syncthreads();
    const SplitChoice choice = shared_choice;
    const int32_t BN = totals->block_n;
    const UnitCosts uc{j.q_begin, j.q_len, j.kv_len, j.shares_kv, j.BM, BN, group, j.head_dim, choice,
                       dkv ? small_block(*totals, choice, j.q_heads, j.kv_heads, j.head_dim, j.compute_units) : 0,
                       dkv && by_item_costs(*totals, choice, j.kv_heads, j.head_dim, j.compute_units)};
    auto unit_of = [&](int32_t i, int32_t &cost, int32_t &parts) {
        if (dkv) uc.dkv(j.dkv_items[i], i, cost, parts);
        else uc.fwd(j.fwd_items[i], NW, cost, parts);
    };
    const int32_t a = first + threadIdx.x / 4, quarter = threadIdx.x % 4;
    int32_t my_cost = 0, my_parts = 0, rank = 0, before = 0, sum = 0;
    if (a < n) unit_of(a, my_cost, my_parts);
    for (int32_t b0 = 0; b0 < n; b0 += 1024) {
        __syncthreads();
        const int32_t lim = min(1024, n - b0);
        for (int32_t i = threadIdx.x; i < ((lim + 15) & ~15); i += blockDim.x) {
            t_cost[i] = -1;
            t_parts[i] = 0;
            if (i < lim) unit_of(b0 + i, t_cost[i], t_parts[i]);
        }
        __syncthreads();
#pragma unroll 2
        for (int32_t x = 4 * quarter; x < lim; x += 16) {
            const int4 c = *(const int4 *)&t_cost[x], p = *(const int4 *)&t_parts[x];
            const int32_t y = b0 + x;
            // ahead of this item: a larger cost, or an equal one and earlier in the list
            rank += (c.x >= my_cost + (y >= a) ? p.x : 0) + (c.y >= my_cost + (y + 1 >= a) ? p.y : 0) +
                    (c.z >= my_cost + (y + 2 >= a) ? p.z : 0) + (c.w >= my_cost + (y + 3 >= a) ? p.w : 0);
            before += (y < a ? p.x : 0) + (y + 1 < a ? p.y : 0) + (y + 2 < a ? p.z : 0) + (y + 3 < a ? p.w : 0);
            sum += p.x + p.y + p.z + p.w;
        }
    }
    rank += __shfl_xor(rank, 1, 64);
    rank += __shfl_xor(rank, 2, 64);
    before += __shfl_xor(before, 1, 64);
    before += __shfl_xor(before, 2, 64);
    sum += __shfl_xor(sum, 1, 64);
    sum += __shfl_xor(sum, 2, 64);
    if (dkv && (int64_t)sum * j.kv_heads * (BN == 256 ? 2 : 1) <= j.compute_units) rank = before;
    if (a < n && dkv) {
        const int4 it = j.dkv_items[a];
        for (int32_t p = quarter; p < my_parts; p += 4) j.dkv_units[rank + p] = make_int4(it.x, it.y, a | p << SKRULL_UNIT_SHIFT, my_parts);
    } else if (a < n) {
        for (int32_t p = quarter; p < my_parts; p += 4) units[rank + p] = a | p << SKRULL_UNIT_SHIFT;
    }
    if (NW == 12 && first == 0) {
        int64_t load = 0;
        int32_t longest = 0, longest_full = 0;
        for (int32_t i = threadIdx.x; i < n; i += blockDim.x) {
            int32_t cost, parts;
            unit_of(i, cost, parts);
            load += (int64_t)parts * (cost + 16);
            longest = max(longest, cost + 16);
            if (uc.more_than_four_blocks(j.fwd_items[i])) longest_full = max(longest_full, cost + 16);
        }
        load = wave_sum(load);
        longest = wave_max(longest);
        longest_full = wave_max(longest_full);
        if ((threadIdx.x & 63) == 0) {  // (zeroed by the ranges kernel)
            atomicAdd((unsigned long long *)&totals->fwd_load, (unsigned long long)load);
            atomicMax(&totals->fwd_longest, longest);
            atomicMax(&totals->fwd_longest_full, longest_full);
        }
    }
    if (first == 0 && threadIdx.x == 0) *(dkv ? &totals->n_dkv_units : &totals->n_units[blockIdx.y - 1]) = sum;
}

// ---------------------------------------------------------------------------
// The whole plan of a small micro-batch in one workgroup: what the four kernels above write, with everything
// in between in LDS.  A plan is a chain of small dependent steps that nothing overlaps: four launches, a copy in, a
// copy out and scratch memory around them took most of its time.  The input is read from pinned host memory
// and the totals are written there.  The call (without destroying the plan) by the several kernels and this
// way: 3 sequences 44 and 34 us, 20 sequences with 91 and 115 items 51 and 39, 64 with 167 and 215 items 53 and 46 (the
// ranks are quadratic: for the line see skrull_attn_plan).
// ---------------------------------------------------------------------------
constexpr int kSmallThreads = SKRULL_SMALL_PLAN, kSmallWaves = kSmallThreads / 64;

// Exclusive scans of N values per thread over the workgroup, and their totals.
template <int N>
__device__ inline void scan_all(const int32_t (&v)[N], int32_t (&excl)[N], int32_t (&total)[N], int32_t (*lds)[kSmallWaves])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t incl[N];
    for (int i = 0; i < N; ++i) incl[i] = v[i];
    for (int off = 1; off < 64; off <<= 1)
        for (int i = 0; i < N; ++i) {
            const int32_t up = __shfl_up(incl[i], off, 64);
            if (lane >= off) incl[i] += up;
        }
    __syncthreads();  // (the last scan's totals have been read)
    if (lane == 63)
        for (int i = 0; i < N; ++i) lds[i][wave] = incl[i];
    __syncthreads();
    for (int i = 0; i < N; ++i) {
        int32_t before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kSmallWaves; w += 4) {
            const int4 x = *(const int4 *)&lds[i][w];
            before += (w < wave ? x.x : 0) + (w + 1 < wave ? x.y : 0) + (w + 2 < wave ? x.z : 0) + (w + 3 < wave ? x.w : 0);
            all += x.x + x.y + x.z + x.w;
        }
        excl[i] = before + incl[i] - v[i];
        total[i] = all;
    }
}

// Position of item `a` of `n` in the stable order of descending cost (costs padded with -1 to a multiple of
// 16); 1 << log_t neighbouring threads, this one being `sub` of them, share an item.
__device__ inline int32_t rank_in(const int32_t *costs, int32_t n, int32_t a, int32_t sub, int32_t log_t)
{
    const int32_t mine = costs[a];
    int32_t rank = 0;
    for (int32_t x = 16 * sub; x < n; x += 16 << log_t) {
        int4 c[4];  // (four reads under way: one at a time, each took the latency of the LDS)
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = *(const int4 *)&costs[x + 4 * i];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int32_t y = x + 4 * i;
            rank += (c[i].x >= mine + (y >= a)) + (c[i].y >= mine + (y + 1 >= a)) + (c[i].z >= mine + (y + 2 >= a)) + (c[i].w >= mine + (y + 3 >= a));
        }
    }
    if (log_t > 0) rank += __shfl_xor(rank, 1, 64);
    if (log_t > 1) rank += __shfl_xor(rank, 2, 64);
    return rank;
}

__global__ __launch_bounds__(kSmallThreads) void plan_small_kernel(SmallPlan j)
{
    __shared__ __align__(16) int32_t q_begin[kSmallThreads + 1], q_len[kSmallThreads + 1], kv_len[kSmallThreads + 1], cu_q[kSmallThreads + 1];
    __shared__ __align__(16) int32_t shares[kSmallThreads + 1], fwd_off[kSmallThreads + 1], dkv_off[kSmallThreads + 1], alt_off[kSmallThreads + 1];
    __shared__ __align__(16) int4 fwd[kSmallThreads], dkv[kSmallThreads];
    __shared__ __align__(16) int32_t cost_f[kSmallThreads], cost_d[kSmallThreads], at[4][kSmallThreads], order[2][kSmallThreads];
    __shared__ __align__(16) int32_t scans[6][kSmallWaves];
    __shared__ int32_t first_bad, longest_s, cost_max;
    __shared__ unsigned long long sum_s, pairs_s, load_s;
    __shared__ PlanTotals tot;
    __shared__ ChainCounts chains;
    const int t = threadIdx.x;
    clear_sets(j.sets);
    const int32_t group = j.q_heads / j.kv_heads, log_bm = __ffs(j.BM) - 1;  // (BM is a power of two)
    if (t == 0) {
        first_bad = 0x7fffffff;
        longest_s = cost_max = 0;
        sum_s = pairs_s = load_s = 0;
    }
    for (int i = t; i < (int)(sizeof tot / 4); i += kSmallThreads) ((int32_t *)&tot)[i] = 0;
    // --- ranges of the sequences' segments
    int32_t qb[2] = {0, 0}, qe[2] = {0, 0}, nseg = 0;
    int64_t pr = 0;
    bool bad = false;
    if (t < j.K) {
        const int32_t s = j.in[t], n = j.in[j.stride + t], r = j.in[2 * j.stride + t], z = j.in[3 * j.stride + t];
        const int64_t chunks = (int64_t)n * (z ? 2 : 1);
        bad = s < 1 || n < 1 || r < 0 || r >= n || (z != 0 && z != 1) || chunks > s;
        if (!bad) {
            nseg = z + 1;
            const int64_t idx[2] = {r, 2 * (int64_t)n - 1 - r};
            for (int part = 0; part < nseg; ++part) {
                qb[part] = chunks == 1 ? 0 : (int32_t)((idx[part] * s) / chunks);
                qe[part] = chunks == 1 ? s : (int32_t)(((idx[part] + 1) * s) / chunks);
                pr += ((int64_t)qe[part] * (qe[part] + 1) - (int64_t)qb[part] * (qb[part] + 1)) / 2;
            }
        }
    }
    const int32_t end = nseg ? qe[nseg - 1] : 0;
    if (nseg) bad = qe[0] - qb[0] + qe[1] - qb[1] > j.max_q_rows || end > j.max_k_rows;
    __syncthreads();
    if (bad) atomicMin(&first_bad, t);
    // --- offsets, for both sizes of key blocks that may be taken
    int32_t nf[2];
    for (int part = 0; part < 2; ++part) nf[part] = (qe[part] - qb[part] + j.BM - 1) >> log_bm;
    const int32_t bn_alt = j.bn_alt ? j.bn_alt : j.BN;
    const int32_t v[6] = {nseg, qe[0] - qb[0] + qe[1] - qb[1], end, nf[0] + nf[1], (int32_t)((uint32_t)(end + j.BN - 1) / (uint32_t)j.BN),
                          (int32_t)((uint32_t)(end + bn_alt - 1) / (uint32_t)bn_alt)};
    int32_t e[6], n_all[6];
    scan_all<6>(v, e, n_all, scans);
    for (int part = 0; part < nseg; ++part) {
        const int32_t sg = e[0] + part;
        j.q_begin[sg] = q_begin[sg] = qb[part];
        j.q_len[sg] = q_len[sg] = qe[part] - qb[part];
        j.kv_len[sg] = kv_len[sg] = qe[part];
        j.cu_q[sg] = cu_q[sg] = e[1] + (part ? qe[0] - qb[0] : 0);
        j.cu_k[sg] = e[2];
        j.shares_kv[sg] = shares[sg] = part;
        fwd_off[sg] = e[3] + (part ? nf[0] : 0);
        dkv_off[sg] = e[4];
        alt_off[sg] = e[5];
    }
    pr = wave_sum(pr);
    const int32_t longest_end = wave_max(end);
    if ((t & 63) == 0) {
        atomicAdd(&pairs_s, (unsigned long long)pr);
        atomicMax(&longest_s, longest_end);
    }
    const int32_t NS = n_all[0], n_fwd = min(n_all[3], j.cap_fwd);
    if (t == 0) {
        j.cu_q[NS] = n_all[1];
        j.cu_k[NS] = n_all[2];
        fwd_off[NS] = n_all[3];
        dkv_off[NS] = n_all[4];
        alt_off[NS] = n_all[5];
    }
    __syncthreads();
    // --- items and their costs, as in plan_emit_kernel
    int4 f = make_int4(0, 0, 0, -1), d = make_int4(0, 0, 0, -1);
    // dK/dV item `i` for key blocks of `bn` rows, whose offsets are `off`
    auto key_item = [&](const int32_t *off, int32_t bn, int32_t i) {
        const int32_t k = owner_of(off, NS, i), b = i - off[k], m0 = max(b * bn - q_begin[k], 0) >> log_bm;
        int32_t cost = ((q_len[k] - 1) >> log_bm) + 1 - m0;
        if (shares[k] && b * bn < kv_len[k - 1]) cost += ((q_len[k - 1] - 1) >> log_bm) + 1 - (max(b * bn - q_begin[k - 1], 0) >> log_bm);
        return make_int4(k, b, m0, cost);
    };
    // sum and maximum of the items' costs
    auto add_costs = [&]() {
        const int64_t c_sum = wave_sum(max(d.w, 0));
        const int32_t c_max = wave_max(d.w);
        if ((t & 63) == 0 && c_sum > 0) {
            atomicAdd(&sum_s, (unsigned long long)c_sum);
            atomicMax(&cost_max, c_max);
        }
        __syncthreads();
    };
    int32_t BN = j.BN, n_dkv = min(n_all[4], j.cap_dkv);
    if (t < n_dkv) d = key_item(dkv_off, BN, t);
    add_costs();
    if (j.bn_alt != 0 &&
        larger_key_blocks((int64_t)sum_s, cost_max, n_all[5], longest_s, j.bn_alt, j.kv_heads, j.compute_units)) {
        BN = j.bn_alt;
        n_dkv = min(n_all[5], j.cap_dkv);
        d = make_int4(0, 0, 0, -1);
        if (t < n_dkv) d = key_item(alt_off, BN, t);
        __syncthreads();
        if (t == 0) {
            sum_s = 0;
            cost_max = 0;
        }
        __syncthreads();
        add_costs();
    }
    if (t < n_fwd) {
        const int32_t k = owner_of(fwd_off, NS, t), m = t - fwd_off[k], row0 = m << log_bm;
        f = make_int4(k, m, cu_q[k] + row0, (int32_t)((uint32_t)(q_begin[k] + row0 + min(q_len[k] - row0, j.BM) + BN - 1) / (uint32_t)BN));
    }
    fwd[t] = f;
    dkv[t] = d;
    cost_f[t] = f.w;
    cost_d[t] = d.w;
    // --- sorted lists
    if (t == 0) {
        tot.total_q = n_all[1];
        tot.total_k = n_all[2];
        tot.n_fwd = n_all[3];
        tot.n_dkv = BN == j.BN ? n_all[4] : n_all[5];
        tot.pairs = (int64_t)pairs_s;
        tot.bad_entry = first_bad == 0x7fffffff ? 0 : first_bad + 1;
        tot.n_seg = NS;
        tot.dkv_cost_sum = sum_s;
        tot.dkv_cost_max = cost_max;
        tot.cap_fwd = j.cap_fwd;
        tot.cap_dkv = j.cap_dkv;
        tot.block_n = BN;
    }
    __syncthreads();
    chains.begin(&tot, j.q_heads, j.head_dim, j.compute_units);
    const int32_t log_t = max(n_fwd, n_dkv) <= kSmallThreads / 4 ? 2 : (max(n_fwd, n_dkv) <= kSmallThreads / 2 ? 1 : 0);
    const int32_t a = t >> log_t, sub = t & ((1 << log_t) - 1);  // threads of an item
    f = fwd[a];
    d = dkv[a];
    const int32_t at_f = rank_in(cost_f, n_fwd, a, sub, log_t), at_d = rank_in(cost_d, n_dkv, a, sub, log_t);
    __syncthreads();
    if (a < n_fwd && sub == 0) {
        fwd[at_f] = f;
        ((int4 *)j.fwd_items)[at_f] = f;
    }
    if (a < n_dkv && sub == (1 << log_t) - 1) {
        dkv[at_d] = d;
        ((int4 *)j.dkv_items)[at_d] = d;
        chains.count(d.w, group);
    }
    __syncthreads();
    chains.end(&tot);
    __syncthreads();
    // --- work units, as in plan_units_kernel
    if (t == 0) tot.split = choose_split(j.asked, tot, j.q_heads, j.kv_heads, j.head_dim, j.longest_seq, j.compute_units);
    __syncthreads();
    const UnitCosts uc{q_begin, q_len, kv_len, shares, j.BM, BN, group, j.head_dim, tot.split,
                       small_block(tot, tot.split, j.q_heads, j.kv_heads, j.head_dim, j.compute_units),
                       by_item_costs(tot, tot.split, j.kv_heads, j.head_dim, j.compute_units)};
    int32_t parts[4] = {0, 0, 0, 0}, cf = -1, cd = -1;  // dK/dV, then 4, 8 and 12 waves
    if (t < n_dkv) uc.dkv(dkv[t], t, cd, parts[0]);
    if (t < n_fwd)
        for (int i = 0; i < SKRULL_UNIT_LISTS; ++i) uc.fwd(fwd[t], 4 * (i + 1), cf, parts[1 + i]);
    cost_f[t] = cf;
    cost_d[t] = cd;
    {
        const int64_t load = wave_sum(t < n_fwd ? (int64_t)parts[3] * (cf + 16) : 0);
        const int32_t longest = wave_max(t < n_fwd ? cf + 16 : 0);
        const int32_t longest_full = wave_max(t < n_fwd && uc.more_than_four_blocks(fwd[t]) ? cf + 16 : 0);
        if ((t & 63) == 0) {
            atomicAdd(&load_s, (unsigned long long)load);
            atomicMax(&tot.fwd_longest, longest);
            atomicMax(&tot.fwd_longest_full, longest_full);
        }
    }
    int32_t ex[4], sum[4];
    scan_all<4>(parts, ex, sum, scans);  // (its barriers also make the costs visible)
    const bool list_order = (int64_t)sum[0] * j.kv_heads * (BN == 256 ? 2 : 1) <= j.compute_units;
    if (sub == 0) {
        order[0][a] = a;
        order[1][a] = a;
    }
    const int32_t by_rounds = rank_in(cost_d, n_dkv, a, sub, log_t), by_keys = rank_in(cost_f, n_fwd, a, sub, log_t);
    if (sub == 0 && a < n_dkv && !list_order) order[0][a] = by_rounds;
    if (sub == 0 && a < n_fwd && j.head_dim == 64) order[1][a] = by_keys;
    if (log_t > 0 && t >= kSmallThreads >> log_t) order[0][t] = order[1][t] = t;
    __syncthreads();
    const int32_t rd = order[0][t], rf = order[1][t];
    at[0][rd] = parts[0];
    for (int i = 1; i < 4; ++i) at[i][rf] = parts[i];
    __syncthreads();
    for (int i = 0; i < 4; ++i) parts[i] = at[i][t];
    scan_all<4>(parts, ex, sum, scans);
    for (int i = 0; i < 4; ++i) at[i][t] = ex[i];
    __syncthreads();
    if (t < n_dkv && j.dkv_units) {
        int32_t c, n;
        uc.dkv(dkv[t], t, c, n);
        for (int32_t p = 0; p < n; ++p) j.dkv_units[at[0][rd] + p] = make_int4(dkv[t].x, dkv[t].y, t | p << SKRULL_UNIT_SHIFT, n);
    }
    if (t < n_fwd)
        for (int i = 0; i < SKRULL_UNIT_LISTS; ++i) {
            int32_t c, n;
            uc.fwd(fwd[t], 4 * (i + 1), c, n);
            if (j.units[i])
                for (int32_t p = 0; p < n; ++p) j.units[i][at[1 + i][rf] + p] = t | p << SKRULL_UNIT_SHIFT;
        }
    if (t == 0) {
        tot.n_dkv_units = j.dkv_units ? sum[0] : 0;
        for (int i = 0; i < SKRULL_UNIT_LISTS; ++i) tot.n_units[i] = j.units[i] ? sum[1 + i] : 0;
        tot.fwd_load = j.units[2] ? (int64_t)load_s : 0;
        if (!j.units[2]) tot.fwd_longest = tot.fwd_longest_full = 0;
    }
    __syncthreads();
    for (int i = t; i < (int)(sizeof tot / 4); i += kSmallThreads) ((int32_t *)j.totals)[i] = ((const int32_t *)&tot)[i];
}

// ---------------------------------------------------------------------------
// Long lists: stable least-significant-digit radix sort on key = key_max - cost
// (ascending key = descending cost), 8 bits per pass, 1024 consecutive items per
// block.  Three kernels per pass: per-block digit histogram; exclusive scan of the
// (digit, block) table in digit-major order; scatter, in which an item's offset is
// its digit's start + the items of that digit in earlier blocks + those before it
// in its own block (which keeps equal keys in their order: the sort is stable).
// ---------------------------------------------------------------------------
constexpr int kRadixBlock = 1024;

__device__ inline int32_t list_length(const PlanTotals *totals, int which)
{
    return which == 0 ? (int32_t)min((long long)totals->n_fwd, (long long)totals->cap_fwd)
                      : (int32_t)min((long long)totals->n_dkv, (long long)totals->cap_dkv);
}

__global__ __launch_bounds__(256) void radix_hist_kernel(const int4 *__restrict__ in, PlanTotals *totals, int which,
                                                         int32_t group, int32_t q_heads, int32_t head_dim,
                                                         int32_t compute_units,
                                                         int32_t key_max, int shift, int32_t nb,
                                                         int32_t *__restrict__ hist)
{
    __shared__ int32_t h[256];
    __shared__ ChainCounts chains;
    const int32_t n = list_length(totals, which);
    const bool counts = which == 1 && shift == 0;
    h[threadIdx.x] = 0;
    if (counts) chains.begin(totals, q_heads, head_dim, compute_units);
    __syncthreads();
    const int32_t base = blockIdx.x * kRadixBlock;
    for (int32_t i = threadIdx.x; i < kRadixBlock; i += 256)
        if (base + i < n) {
            const int32_t cost = in[base + i].w;
            atomicAdd(&h[((key_max - cost) >> shift) & 255], 1);
            if (counts) chains.count(cost, group);
        }
    __syncthreads();
    if (counts) chains.end(totals);
    hist[threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// one block; thread d scans the counts of digit d over the blocks, then the digits are scanned
__global__ __launch_bounds__(256) void radix_scan_kernel(int32_t *__restrict__ hist, int32_t nb)
{
    __shared__ int64_t lds[kScanThreads];
    const int d = threadIdx.x;
    int32_t run = 0;
    for (int32_t b = 0; b < nb; ++b) {
        const int32_t c = hist[d * nb + b];
        hist[d * nb + b] = run;
        run += c;
    }
    int64_t tot;
    const int32_t start = (int32_t)block_exclusive_scan(run, lds, &tot);
    for (int32_t b = 0; b < nb; ++b) hist[d * nb + b] += start;
}

__global__ __launch_bounds__(256) void radix_scatter_kernel(const int4 *__restrict__ in,
                                                            const PlanTotals *__restrict__ totals, int which,
                                                            int32_t key_max, int shift, int32_t nb,
                                                            const int32_t *__restrict__ hist,
                                                            int4 *__restrict__ out)
{
    __shared__ unsigned char dig[kRadixBlock];
    const int32_t n = list_length(totals, which);
    const int32_t base = blockIdx.x * kRadixBlock;
    const int32_t cnt = min(kRadixBlock, n - base);
    if (cnt <= 0) return;
    // thread t owns the consecutive items 4t .. 4t+3 of the block
    int4 mine[4];
    for (int e = 0; e < 4; ++e) {
        const int32_t i = 4 * threadIdx.x + e;
        if (i < cnt) {
            mine[e] = in[base + i];
            dig[i] = (unsigned char)(((key_max - mine[e].w) >> shift) & 255);
        }
    }
    __syncthreads();
    for (int e = 0; e < 4; ++e) {
        const int32_t i = 4 * threadIdx.x + e;
        if (i >= cnt) break;
        const unsigned char d = dig[i];
        int32_t before = 0;  // items of the same digit earlier in this block
        for (int32_t j = 0; j < i; ++j) before += dig[j] == d;
        out[hist[(int32_t)d * nb + blockIdx.x] + before] = mine[e];
    }
}

}  // namespace

hipError_t launch_plan_ranges(const int32_t *S, const int32_t *N, const int32_t *r,
                              const int32_t *cut, int32_t K, int32_t BM, int32_t BN,
                              int32_t max_q_rows, int32_t max_k_rows, int32_t *q_begin,
                              int32_t *q_len, int32_t *kv_len, int32_t *cu_q, int32_t *cu_k,
                              int32_t *shares_kv, int32_t *fwd_off, int32_t *dkv_off,
                              int32_t cap_fwd, int32_t cap_dkv, int32_t bn_alt, int32_t kv_heads,
                              int32_t compute_units, PlanTotals *totals, hipStream_t st)
{
    plan_ranges_kernel<<<1, kScanThreads, 0, st>>>(S, N, r, cut, K, BM, BN, max_q_rows, max_k_rows,
                                                   q_begin, q_len, kv_len, cu_q, cu_k, shares_kv,
                                                   fwd_off, dkv_off, cap_fwd, cap_dkv, bn_alt, kv_heads,
                                                   compute_units, totals);
    return hipGetLastError();
}

// Above this many items (the host's upper bound) a list is sorted by radix passes instead of
// by rank counting, which is quadratic: both lists together take 14 us at 1,318 items of dK/dV and 18 at 1,982; one
// radix pass takes 73 us at 2,673.  (The line could lie higher, but the lists of units hold an item's
// position in SKRULL_UNIT_SHIFT bits.)
constexpr int32_t kRankSortMax = 1 << SKRULL_UNIT_SHIFT;

int plan_radix_passes(int32_t cap, int32_t cost_bound)
{
    if (cap <= kRankSortMax) return 0;
    int bits = 1;
    while (bits < 31 && (1 << bits) <= cost_bound) ++bits;
    return (bits + 7) / 8;
}

int64_t plan_unit_ints(const skrull_attn_plan_t *p, int32_t cap_fwd, int which)
{
    const int waves = 4 * (which + 1);
    if (cap_fwd > kRankSortMax || p->Hq > SKRULL_UNIT_HEADS || (waves == 12 && p->d != 64)) return 0;
    return (int64_t)cap_fwd * ((p->BM / 32 * (p->Hq / p->Hkv) + waves - 1) / waves);
}

int64_t plan_radix_ints(int32_t cap_fwd, int32_t cap_dkv, int32_t cost_bound)
{
    int64_t n = 0;
    if (plan_radix_passes(cap_fwd, cost_bound)) n += 256 * (int64_t)((cap_fwd + kRadixBlock - 1) / kRadixBlock);
    if (plan_radix_passes(cap_dkv, cost_bound)) n += 256 * (int64_t)((cap_dkv + kRadixBlock - 1) / kRadixBlock);
    return n;
}

// Radix sort of one list.  `a` holds the emitted items when the number of passes is odd, `b`
// when it is even, so that the last pass always writes the plan's array `b`.
static hipError_t radix_sort_list(const skrull_attn_plan_t *p, int which, int32_t cap, int passes, int32_t compute_units,
                                  int4 *a, int4 *b, int32_t *hist, PlanTotals *totals, hipStream_t st)
{
    const int32_t group = p->Hq / p->Hkv;
    int key_bits = 8 * passes;
    const int32_t key_max = key_bits >= 31 ? INT32_MAX : (1 << key_bits) - 1;  // >= any cost
    const int32_t nb = (cap + kRadixBlock - 1) / kRadixBlock;
    int4 *src = (passes & 1) ? a : b, *dst = (passes & 1) ? b : a;
    for (int pass = 0; pass < passes; ++pass) {
        radix_hist_kernel<<<nb, 256, 0, st>>>(src, totals, which, group, p->Hq, p->d, compute_units, key_max, 8 * pass, nb, hist);
        radix_scan_kernel<<<1, 256, 0, st>>>(hist, nb);
        radix_scatter_kernel<<<nb, 256, 0, st>>>(src, totals, which, key_max, 8 * pass, nb, hist, dst);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        int4 *t = src; src = dst; dst = t;
    }
    return hipSuccess;
}

hipError_t launch_plan_items(const skrull_attn_plan_t *p, const int32_t *fwd_off,
                             const int32_t *dkv_off, int32_t cap_fwd, int32_t cap_dkv,
                             int32_t *scratch_fwd, int32_t *scratch_dkv, int32_t *radix_hist,
                             int32_t cost_bound, int32_t compute_units, PlanTotals *totals, hipStream_t st)
{
    // grids are sized by the host's upper bounds of the item counts; the kernels take the
    // counts from `totals` on the device, so no round trip to the host is needed in between
    const int32_t n = cap_fwd > cap_dkv ? cap_fwd : cap_dkv;
    // the emit kernel writes each list where its sort starts from
    const int passes_f = plan_radix_passes(cap_fwd, cost_bound), passes_d = plan_radix_passes(cap_dkv, cost_bound);
    const bool fwd_even = passes_f != 0 && passes_f % 2 == 0, dkv_even = passes_d != 0 && passes_d % 2 == 0;
    plan_emit_kernel<<<(n + 255) / 256, 256, 0, st>>>(
        p->NS, p->BM, p->q_begin, p->q_len, p->kv_len, p->cu_q, p->shares_kv, fwd_off, dkv_off,
        (int4 *)(fwd_even ? p->fwd_items : scratch_fwd), (int4 *)(dkv_even ? p->dkv_items : scratch_dkv), totals,
        (int4 *)p->sets);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // short lists by rank counting, both in one launch when both are short
    if (passes_f == 0 || passes_d == 0) {
        const int first = passes_f == 0 ? 0 : 1, lists = (passes_f == 0) + (passes_d == 0);
        const int32_t most = passes_f == 0 && passes_d == 0 ? n : (passes_f == 0 ? cap_fwd : cap_dkv);
        plan_sort_kernel<<<dim3((most + kSortItems - 1) / kSortItems, lists), 256, 0, st>>>(
            SortJob{(const int4 *)scratch_fwd, (int4 *)p->fwd_items}, SortJob{(const int4 *)scratch_dkv, (int4 *)p->dkv_items},
            first, totals, p->Hq / p->Hkv, p->Hq, p->d, compute_units);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    int32_t *hist_dkv = radix_hist;
    if (passes_f) hist_dkv += 256 * (int64_t)((cap_fwd + kRadixBlock - 1) / kRadixBlock);
    if (passes_f) {
        e = radix_sort_list(p, 0, cap_fwd, passes_f, compute_units, (int4 *)scratch_fwd, (int4 *)p->fwd_items, radix_hist, totals, st);
        if (e != hipSuccess) return e;
    }
    if (passes_d) e = radix_sort_list(p, 1, cap_dkv, passes_d, compute_units, (int4 *)scratch_dkv, (int4 *)p->dkv_items, hist_dkv, totals, st);
    return e;
}

int64_t plan_dkv_unit_ints(const skrull_attn_plan_t *p, int32_t asked, int32_t cap_dkv)
{
    const int32_t group = p->Hq / p->Hkv, parts = asked ? asked : (group > kMaxParts ? group : kMaxParts);
    if (cap_dkv > kRankSortMax || p->Hq > SKRULL_UNIT_HEADS) return 0;
    return 4 * (int64_t)cap_dkv * parts;
}

hipError_t launch_plan_units(const skrull_attn_plan_t *p, int32_t asked, int32_t longest_seq, int32_t cap_fwd, int32_t cap_dkv,
                             int32_t compute_units, PlanTotals *totals, hipStream_t st)
{
    const int32_t f = p->units[0] ? cap_fwd : 1, d = p->dkv_units ? cap_dkv : 1, most = f > d ? f : d;
    plan_units_kernel<<<dim3((most + kSortItems - 1) / kSortItems, p->units[0] ? 1 + SKRULL_UNIT_LISTS : 1), 256, 0, st>>>(
        UnitsJob{(const int4 *)p->fwd_items, (const int4 *)p->dkv_items, p->q_begin, p->q_len, p->kv_len, p->shares_kv, p->BM, p->Hq,
                 p->Hkv, p->d, asked, longest_seq, compute_units, {p->units[0], p->units[1], p->units[2]}, p->dkv_units},
        totals);
    return hipGetLastError();
}

hipError_t launch_plan_small(const SmallPlan &job, hipStream_t st)
{
    plan_small_kernel<<<1, kSmallThreads, 0, st>>>(job);
    return hipGetLastError();
}
