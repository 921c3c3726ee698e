// Backward kernels: D = rowsum(dO * O), dQ, and dK/dV with the GQA head
// reduction, for the packed varlen causal attention of fwd.hip.
//
//   P_ij  = exp(scale * q_i.k_j - LSE_i)          dP_ij = dO_i . v_j
//   dS_ij = P_ij (dP_ij - D_i)
//   dQ_i  = scale * sum_j dS_ij k_j
//   dK_j  = scale * sum_{h in group} sum_i dS_ij q_i
//   dV_j  =         sum_{h in group} sum_i P_ij dO_i
//
// dQ kernel: work items, workgroup shape and orientation of the forward kernel
// (query index on the MFMA column, so LSE_i and D_i are per-lane scalars):
//     S^T = K Q^T, dP^T = V dO^T           A = K / V tile rows (LDS), B = Q / dO (registers)
//     dQ^T[t,i] += sum_j K^T[t,j] dS^T[j,i] A = transposed K tile (LDS), B = dS^T (registers)
// dK/dV kernel: one workgroup owns BN key rows of one KV head and walks over
// the g query heads of the group and the query tiles that can see them; the
// key index is on the MFMA column, so the two accumulators of a lane belong to
// one key row and the group sum never leaves registers:
//     S = Q K^T, dP = dO V^T               A = Q / dO tile rows (LDS), B = K / V (registers)
//     dV^T[t,j] += sum_i dO^T[t,i] P[i,j]   A = transposed dO tile (LDS), B = P (registers)
//     dK^T[t,j] += sum_i Q^T[t,i] dS[i,j]   A = transposed Q tile (LDS),  B = dS (registers)
// The paper's FLOPs model counts this quadratic work per sequence (App. B.2);
// the work-list order balances it over compute units (plan.hip).
#include <type_traits>

#include "common.h"
#include "mfma.h"
#include "queue.h"
#include "tiles.h"

namespace {

constexpr float kLog2e = 1.4426950408889634f;

// How a dK/dV work index stands for an item, a part of its chain, a KV head and a pass over the item's
// key rows; quotients as in RowMap.  With a list of units these go out in its order.  Without one (lists too
// long for the rank sort, very many heads) handed out first are `n_whole_first` items that one workgroup does
// whole, then the parts of the first `n_split` items of the list, then the rest: the units of all
// three run from long to short, and the whole items of the middle are as long as the longest parts.
struct KeyMap {
    int32_t BN, g, passes, Hkv;                 // query heads per KV head; workgroups per (item, part, KV head)
    int32_t n_split, n_whole_first, parts, chain;  // see skrull_attn_plan
    int32_t part_rows;                          // rows of one part's partial sums; 0: the rows of K themselves
    uint64_t inv_passes, inv_hkv;
    const int4 *units;                          // null, or the work units (skrull_attn_plan::dkv_units)
    uint64_t inv_whole;
};
// workgroups that share an item of the first n_split
__device__ __forceinline__ int parts_of(const KeyMap &m, int cost)
{
    return m.chain == 0 ? m.parts : min(m.parts, (cost * m.g + m.chain - 1) / m.chain);
}

struct BwdParams {
    const uint16_t *q, *k, *v, *d_o, *o;
    const float *lse;
    float *delta, *lse2;  // workspace [Hq, total_q] each: -D and LSE * log2(e), written by the dQ kernel
    uint16_t *dq, *dk, *dv;
    const int4 *fwd_items, *dkv_items;
    const int32_t *cu_q, *cu_k, *q_begin, *q_len, *kv_len, *shares_kv;
    RowMap rows;  // dQ: which row blocks a workgroup's waves take
    KeyMap keys;  // dK/dV: which keys and heads a workgroup takes
    int32_t Hq, Hkv, total_q;
    float scale, scale_log2;
    // workgroups that share a dK/dV item leave unrounded partial sums in dk_part / dv_part
    // ([part][row][Hkv][D] fp32) for dkv_reduce_kernel
    int32_t total_k;
    float *dk_part, *dv_part;
    WgTrace *trace_dq, *trace_dkv;  // null, or one record per work item (measurement aid)
    WorkQueue *queue_dq, *queue_dkv;  // work queues of the persistent launches, zero when they start
    int32_t queue_stride;             // their dies' distance
    int32_t n_work_dq, n_work_dkv;    // work items: what a plain grid would have as workgroups
    int32_t *clear;                   // null, or what the stream's next call will use: zeroed by this one (see DefaultStream)
    // one launch for all: dQ work items whose -D and LSE dK/dV may read; parts of shared dK/dV items whose sums are
    // stored, of each (item, KV head) or, for very many of these, of all of them; pieces of the sums of these that have been handed out
    int32_t *rows_ready, *parts_stored, *next_sum;
    int32_t n_parts;                  // work items that are parts of shared dK/dV items; 0: they are counted for each item
};

// ---------------------------------------------------------------------------
// dQ
// ---------------------------------------------------------------------------
// The dQ kernel comes in three shapes, like the forward, and the small one in two kinds.  Large: 8 wavefronts (256 query rows), two per SIMD, with a
// five-slot K ring and a four-slot V ring, and a software pipeline from one half tile of keys to the next,
// which takes 191 registers at head_dim 64 and 254 at 128.  At head_dim 64 also two that do one half tile
// after another: with nothing kept from one to the next 168 registers do, so that three wavefronts per SIMD overlap
// with each other instead.  Wide: 12 wavefronts, K and V rings of four slots; small: workgroups of 4
// wavefronts, rings of two slots, a barrier per tile.  A wavefront alone on its SIMD is slower this way and
// eight are as fast (23,053 tokens, 16/16 heads: backward 785 us pipelined, 792 with 8 of 12 at work), so the
// large shape stays where a long unit is what a launch waits for and where 12 cannot be filled, and the small one is
// pipelined too (three K slots, two workgroups per unit) where long units would leave the third place of a unit empty
// (the plan decides by their length and number).
// 26,624 tokens in 64 sequences, 14/2 heads: dQ 94 us large, 86 wide; 32,768 of 16 to 1,024: 88 and 75; slices of
// three long sequences, 1.5e9 triples and more: forward and backward 6,240 with small workgroups that were pipelined (two
// per unit), 6,200 this way (three).
constexpr int NWQ_LARGE = 8, NWQ_SMALL = 4, NWQ_WIDE = 12;

// Two scores and two (dP - D) values -> one packed bf16 pair of dS, in two parts so
// that each part can sit behind one MFMA of a pipelined step (plain arithmetic would
// be moved by the compiler to its first use, behind all the MFMAs of the step).
// Part one: p = exp2(s * c - lse'); part two: p * (dP - D), packed.  Each exponential
// has an instruction between it and the first use of its result.
__device__ __forceinline__ void ds_exp2(float s0, float s1, float c, float l, float &t0, float &t1)
{
    asm volatile("v_fma_f32 %0, %2, %4, -%5\n\t"
                 "v_fma_f32 %1, %3, %4, -%5\n\t"
                 "v_exp_f32 %0, %0\n\t"
                 "v_exp_f32 %1, %1"
                 : "=&v"(t0), "=&v"(t1)
                 : "v"(s0), "v"(s1), "s"(c), "v"(l));
}
__device__ __forceinline__ uint32_t ds_mul_pack(float t0, float t1, float g0, float g1)
{
    uint32_t pk;
    float u0, u1;
    asm volatile("v_mul_f32 %1, %3, %5\n\t"
                 "v_mul_f32 %2, %4, %6\n\t"
                 "v_cvt_pk_bf16_f32 %0, %1, %2"
                 : "=&v"(pk), "=&v"(u0), "=&v"(u1)
                 : "v"(t0), "v"(t1), "v"(g0), "v"(g1));
    return pk;
}

// One workgroup = part of a forward work item (at most 256 query rows) x one KV head (tiles.h:
// row_blocks); each wave owns 32 query rows of one head.  In the large shape K and V stream in
// 64-row tiles through LDS rings (K: five slots, V: four), fetched two tiles ahead by
// buffer loads that write LDS directly; fetches are issued, and the workgroup meets
// at a barrier, every second tile.  Half-tile j (32 keys) goes through
//   A(j): S^T = K Q^T and dP^T - D = V dO^T with -D as the accumulator's start,
//   V(j): dS^T = exp2(S^T c - LSE') (dP^T - D), rounded to bf16,
//   B(j): dQ^T += K^T dS^T,
// and step j issues A(j+1) with the vector work V(j) spread between its MFMAs, then
// B(j).  B(j) reads the transposed K of the half tile BEFORE the one A(j+1) reads,
// which is why the K ring has one slot more than the V ring.  Steps at the start, the
// end and the causal diagonal of a wave's range take a plain path with guards.
// Where the work of dQ (KV: of dK/dV) comes from, read anew each time: kept through the work loops, as the compiler
// would where both are in one kernel, these few values cost it scalar registers (45 spilled instead of 14).
template <bool KV> struct BwdSource {
    __device__ __forceinline__ WorkQueue *queue() const { return KV ? kernarg<BwdParams>()->queue_dkv : kernarg<BwdParams>()->queue_dq; }
    __device__ __forceinline__ int stride() const { return kernarg<BwdParams>()->queue_stride; }
    __device__ __forceinline__ int items() const { return KV ? kernarg<BwdParams>()->n_work_dkv : kernarg<BwdParams>()->n_work_dq; }
};
using DqFeed = WorkFeed<false, BwdSource<false>>;
using DkvFeed = WorkFeed<false, BwdSource<true>>;

// LDS of a dQ workgroup
template <int D, int NWQ, bool PIPED>
struct DqLds {
    static constexpr bool SMALL = NWQ == NWQ_SMALL, WIDE = NWQ == NWQ_WIDE;
    static constexpr int KSL = SMALL ? (PIPED ? 3 : 2) : (WIDE ? 4 : 5), VSL = SMALL ? 2 : 4;  // ring slots
    static constexpr int MORE = (KSL + VSL) * TileGeom<D>::BYTES;                              // what the staging of a wide workgroup takes beside the rings
    static constexpr int BYTES = MORE + (WIDE ? 4 * WaveStage<D>::BYTES : 0);
};

// A word that other workgroups of the launch read.
template <typename T> __device__ __forceinline__ void store_shared(T *p, T x)
{
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void count_one(int32_t *counter)
{
    (void)__hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Does work item `bid`, whose rows are `rb`; returns the next one and leaves its rows in `rb`.
// ONE: dK/dV follows in the same launch, so -D and LSE are stored when they are known, and the item is counted
// as ready once they are in memory.
template <int D, int NWQ, bool PIPED, bool ONE>
__device__ __forceinline__ int dq_work(const int bid, RowBlocks &rb, DqFeed &feed, unsigned char *lds)
{
    const kernarg_t<BwdParams> prm = kernarg<BwdParams>();
    // not PIPED: three wavefronts per SIMD, one half tile after another; PIPED: two
    typedef DqLds<D, NWQ, PIPED> Lds;
    constexpr bool SMALL = Lds::SMALL, WIDE = Lds::WIDE;
    constexpr int KSL = Lds::KSL, VSL = Lds::VSL;
    static_assert(PIPED ? !WIDE : (KSL & (KSL - 1)) == 0, "K tile t in slot t mod KSL");
    constexpr int KS = D / 16, TT = D / 32, KT = TILE_ROWS;
    typedef TileGeom<D> G;
    constexpr int TB = G::BYTES;
    constexpr int HALF = 32 * G::ROWB;  // byte offset of a tile's second 32 rows
    typedef RingLoader<D, NWQ> Loader;
    static_assert(KS == 2 * TT, "B(j) has half as many MFMAs as A(j+1)");

    unsigned char (*lds_k)[TB] = (unsigned char (*)[TB])lds, (*lds_v)[TB] = lds_k + KSL;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, lives in an SGPR
    const int n = lane & 31, h = lane >> 5;
    const int c = rb.c;

    FragAddr<D> fa;
    fa.init(lane);
    Loader ld;
    ld.init(lane, wave, (uint32_t)prm->Hkv * D * 2);
    const uint32_t ring_k = lds_addr(&lds_k[0][0]), ring_v = lds_addr(&lds_v[0][0]);

    const int kvl = rb.kvl, kbase = rb.kbase;
    const uint64_t trace_t0 = trace_begin(prm->trace_dq);
    const int p0 = rb.p0;  // global position of the item's first query
    const int rows = rb.rows, qrow0 = rb.qrow0;
    const int n_tiles = (p0 + min(rb.block(0) * 32 + 32, rows) + KT - 1) / KT;  // for the workgroup's last row block
    const float cs = prm->scale_log2;

    const bool wave_active = rb.has(wave);
    const int wrow0 = wave_active ? rb.block(wave) * 32 : 0;  // first row of this wave's block inside the item
    const int head = rb.head(wave);
    const int my_i = wrow0 + n;
    const int w_pmin = p0 + wrow0;
    const int w_pmax = p0 + min(wrow0 + 31, rows - 1);
    // half tiles (32 keys) of this wave: 0..L hold a visible key, those below n_full only visible keys
    const int L = wave_active ? w_pmax / 32 : -1;
    const int n_full = wave_active ? (w_pmin + 1) / 32 : 0;

    const i32x4 rk = ld.rsrc(prm->k + ((size_t)kbase * prm->Hkv + c) * D, kvl);
    const i32x4 rv = ld.rsrc(prm->v + ((size_t)kbase * prm->Hkv + c) * D, kvl);

    // Large and wide shapes: the fetch group issued at the start of an even period t is K and V tiles
    // t+2, t+3 (tiles past the end read as zero).  Small shape: every period t fetches K
    // and V tile t+1.
    int kslot = 0;  // slot of K tile t (t mod KSL), advanced at the end of every period
    auto fetch = [&](int t) __attribute__((always_inline)) {
        if (SMALL) {
            ld.load(rk, ring_k + (uint32_t)(PIPED ? (kslot == 2 ? 0 : kslot + 1) : (t + 1) & 1) * TB, (t + 1) * KT, wave);
            ld.load(rv, ring_v + (uint32_t)((t + 1) & 1) * TB, (t + 1) * KT, wave);
        } else if (WIDE) {
#pragma unroll
            for (int x = 2; x < 4; ++x) {
                ld.load(rk, ring_k + (uint32_t)((t + x) & 3) * TB, (t + x) * KT, wave);
                ld.load(rv, ring_v + (uint32_t)((t + x) & 3) * TB, (t + x) * KT, wave);
            }
        } else {
            const int k2 = kslot >= 3 ? kslot - 3 : kslot + 2, k3 = kslot >= 2 ? kslot - 2 : kslot + 3;
            ld.load(rk, ring_k + (uint32_t)k2 * TB, (t + 2) * KT, wave);
            ld.load(rv, ring_v + (uint32_t)((t + 2) & 3) * TB, (t + 2) * KT, wave);
            ld.load(rk, ring_k + (uint32_t)k3 * TB, (t + 3) * KT, wave);
            ld.load(rv, ring_v + (uint32_t)((t + 3) & 3) * TB, (t + 3) * KT, wave);
        }
    };
    // start-up: the tiles of the first period(s).  The fetch group of period 0 follows after the
    // barrier below, because until then its slots stage this item's rows of Q, dO and O.
    ld.load(rk, ring_k, 0, wave);
    ld.load(rv, ring_v, 0, wave);
    if (!SMALL) {
        ld.load(rk, ring_k + TB, KT, wave);
        ld.load(rv, ring_v + TB, KT, wave);
    }
    // this wave's staging region: half a ring slot that holds no tile yet (large shape: K slots
    // 2-4 for waves 0-5 and V slots 2-3 for waves 6-7; wide shape: K slots 2-3, V slots 2-3 and a
    // little more; small shape: K slot 1 and V slot 1, or K slots 1-2 of three)
    typedef WaveStage<D> Stage;
    static_assert(2 * Stage::BYTES == TB, "two staging regions per ring slot");
    const uint32_t stage = SMALL ? (PIPED || wave < 2 ? ring_k + TB + (uint32_t)wave * Stage::BYTES : ring_v + TB + (uint32_t)(wave - 2) * Stage::BYTES)
                         : WIDE  ? (wave < 4   ? ring_k + 2 * TB + (uint32_t)wave * Stage::BYTES
                                    : wave < 8 ? ring_v + 2 * TB + (uint32_t)(wave - 4) * Stage::BYTES
                                               : lds_addr(lds + Lds::MORE) + (uint32_t)(wave - 8) * Stage::BYTES)
                                 : (wave < 6 ? ring_k + 2 * TB + (uint32_t)wave * Stage::BYTES
                                             : ring_v + 2 * TB + (uint32_t)(wave - 6) * Stage::BYTES);

    // B operands held for the whole item: this lane's query row of Q and dO
    bf16x8 qf[KS], dof[KS];
    float lse2, nd;
    {
        Stage st;
        st.init(lane);
        const uint32_t pitch = (uint32_t)prm->Hq * D * 2;
        const size_t hoff = ((size_t)qrow0 * prm->Hq + head) * D;
        u32x4 vq[Stage::N], vg[Stage::N], vo[Stage::N];
        st.load(vq, prm->q + hoff, pitch, wrow0, rows);
        st.load(vg, prm->d_o + hoff, pitch, wrow0, rows);
        st.load(vo, prm->o + hoff, pitch, wrow0, rows);
        const int my_row = qrow0 + min(my_i, rows - 1);  // packed row, clamped for loads
        lse2 = prm->lse[(size_t)head * prm->total_q + my_row] * kLog2e;
        st.put(stage, vq);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = fa.rows_at(stage, ks);
        st.put(stage, vg);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) dof[ks] = fa.rows_at(stage, ks);
        st.put(stage, vo);
        // D = rowsum(dO * O) of this lane's row (each half of the wave holds half of the
        // head dims) and LSE in the exp2 domain; both are stored for dK/dV, which takes -D as the start of its dP
        // accumulator: now where that follows in this launch (share_rows), else at the end of the item
        float dsum = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const uint4 ow = __builtin_bit_cast(uint4, fa.rows_at(stage, ks));
            const uint4 gw = __builtin_bit_cast(uint4, dof[ks]);
            const uint32_t a[4] = {ow.x, ow.y, ow.z, ow.w}, b[4] = {gw.x, gw.y, gw.z, gw.w};
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                dsum += __builtin_bit_cast(float, a[w] << 16) * __builtin_bit_cast(float, b[w] << 16);
                dsum += __builtin_bit_cast(float, a[w] & 0xffff0000u) * __builtin_bit_cast(float, b[w] & 0xffff0000u);
            }
        }
        nd = -add_other_half(dsum);
    }
    // ONE: -D and LSE go out now.  The wait for the stores costs an item's start a microsecond, so only the last items,
    // for which others may already be waiting, count themselves here; the others do behind the next barrier.
    const bool last_items = ONE && bid + (int)gridDim.x >= prm->n_work_dq;
    auto share_rows = [&]() __attribute__((always_inline)) {
        if (wave_active && h == 0 && my_i < rows) {
            const kernarg_t<BwdParams> out = kernarg<BwdParams>();
            const size_t at = (size_t)head * out->total_q + qrow0 + my_i;
            store_shared(out->delta + at, nd);
            store_shared(out->lse2 + at, lse2);
        }
    };
    // (behind a barrier before which every wave has waited for its stores)
    auto count_ready = [&]() __attribute__((always_inline)) {
        if (tid == 0) count_one(kernarg<BwdParams>()->rows_ready);
    };
    if (ONE && last_items) share_rows();
    // Everything issued so far has to land here: the compiler's own count of
    // outstanding loads must be zero before the loops, or the waits it places
    // for these fragments would also wait for the tile fetches in flight.
    wait_vmem();
    __syncthreads();
    if (ONE && last_items) count_ready();
    if ((SMALL ? 1 : 2) < n_tiles) fetch(0);  // the staging regions are free again
    if (ONE && !last_items) share_rows();

    f32x16 acc[TT];
    zero_acc(acc);

    // ---- pipelined step j: A(j+1) from kp / vp with V(j) on s_in / g_in between its
    // MFMAs, then B(j) on the transposed K at kt.  FIRST: first step of a period (reads
    // its first operands itself and, at the end, those of the second step from kp2 / vp2);
    // otherwise they are already in fr.
    auto steady = [&](auto first_tag, const unsigned char *kp, const unsigned char *vp,
                      const unsigned char *kt, const unsigned char *kp2, const unsigned char *vp2,
                      const f32x16 &s_in, const f32x16 &g_in, f32x16 &s_out, f32x16 &g_out,
                      bf16x8 (&fr)[4]) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_tag)::value;
        // operand stream of the step: 2*KS reads for A (K rows, V rows alternating), then 2*TT for B
        auto operand = [&](int x) __attribute__((always_inline)) {
            if (x < 2 * KS) return (x & 1) ? fa.rows(vp, 0, x >> 1) : fa.rows(kp, 0, x >> 1);
            const int y = x - 2 * KS;
            return fa.cols(kt, y % TT, y / TT);
        };
        if (FIRST) {
#pragma unroll
            for (int x = 0; x < 3; ++x) fr[x] = operand(x);
        }
        SB();
        uint32_t pw[8];
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            constexpr int EPS = 16 / KS;  // dS values per step of the loop (2 or 4)
            float t[EPS];
            if (i == 0) {
                f32x16 z;
#pragma unroll
                for (int v = 0; v < 16; ++v) z[v] = 0.0f;
                s_out = mfma32(fr[0], qf[0], z);
            } else {
                s_out = mfma32(fr[(2 * i) % 4], qf[i], s_out);
            }
#pragma unroll
            for (int e = 0; e < EPS; e += 2)
                ds_exp2(s_in[EPS * i + e], s_in[EPS * i + e + 1], cs, lse2, t[e], t[e + 1]);
            fr[(2 * i + 3) % 4] = operand(2 * i + 3);
            SB();
            if (i == 0) {
                f32x16 z;
#pragma unroll
                for (int v = 0; v < 16; ++v) z[v] = nd;
                g_out = mfma32(fr[1], dof[0], z);
            } else {
                g_out = mfma32(fr[(2 * i + 1) % 4], dof[i], g_out);
            }
#pragma unroll
            for (int e = 0; e < EPS; e += 2)
                pw[(EPS * i + e) >> 1] = ds_mul_pack(t[e], t[e + 1], g_in[EPS * i + e], g_in[EPS * i + e + 1]);
            fr[(2 * i + 4) % 4] = operand(2 * i + 4);
            SB();
        }
        const bf16x8 ds0 = as_bf16x8(make_uint4(pw[0], pw[1], pw[2], pw[3]));
        const bf16x8 ds1 = as_bf16x8(make_uint4(pw[4], pw[5], pw[6], pw[7]));
#pragma unroll
        for (int y = 0; y < 2 * TT; ++y) {
            acc[y % TT] = mfma32(fr[(2 * KS + y) % 4], y < TT ? ds0 : ds1, acc[y % TT]);
            const int nx = y + 3;  // of this step's B stream, then of the next step's A stream
            if (nx < 2 * TT) {
                fr[(2 * KS + nx) % 4] = operand(2 * KS + nx);
            } else if (FIRST) {
                const int x = nx - 2 * TT;
                fr[x] = (x & 1) ? fa.rows(vp2, 0, x >> 1) : fa.rows(kp2, 0, x >> 1);
            }
            SB();
        }
    };

    // ---- plain step j with run-time guards (start, end and diagonal of the wave's range)
    auto generic = [&](int j, const unsigned char *kp, const unsigned char *vp, const unsigned char *kt,
                       const f32x16 &s_in, const f32x16 &g_in, f32x16 &s_out, f32x16 &g_out)
                       __attribute__((always_inline)) {
        if (j + 1 <= L) {  // A(j+1)
#pragma unroll
            for (int v = 0; v < 16; ++v) { s_out[v] = 0.0f; g_out[v] = nd; }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                s_out = mfma32(fa.rows(kp, 0, ks), qf[ks], s_out);
                g_out = mfma32(fa.rows(vp, 0, ks), dof[ks], g_out);
                if (ks % 4 == 3) SB();
            }
        }
        if (j >= 0 && j <= L) {  // V(j), B(j)
            f32x16 ds;
#pragma unroll
            for (int v = 0; v < 16; ++v) ds[v] = fast_exp2(__builtin_fmaf(s_in[v], cs, -lse2)) * g_in[v];
            if (j >= n_full) {  // half tile touches the diagonal for this wave
                // relative position from an opaque copy of the lane index: the sixteen
                // per-register thresholds are formed here rather than kept for the whole kernel
                int li = lane;
                asm volatile("" : "+v"(li));
                const int rel = p0 + wrow0 + (li & 31) - 32 * j - 4 * (li >> 5);  // my_pos - 32j - 4h
#pragma unroll
                for (int v = 0; v < 16; ++v) ds[v] = (8 * (v >> 2) + (v & 3) > rel) ? 0.0f : ds[v];
            }
            SB();
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const bf16x8 b = acc_to_b(ds, kb);
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) acc[tt] = mfma32(fa.cols(kt, tt, kb), b, acc[tt]);
                SB();
            }
        }
    };

    if constexpr (!PIPED) {
        // Half tile j: A(j), V(j), B(j), nothing kept from one to the next
        auto half = [&](int j, const unsigned char *kp, const unsigned char *vp) __attribute__((always_inline)) {
            bf16x8 fk[KS], fv[KS], ct[2 * TT];
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                fk[i] = fa.rows(kp, 0, i);
                fv[i] = fa.rows(vp, 0, i);
            }
            SB();
            f32x16 s, g;
#pragma unroll
            for (int v = 0; v < 16; ++v) { s[v] = 0.0f; g[v] = nd; }
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                s = mfma32(fk[i], qf[i], s);
                ct[i] = fa.cols(kp, i % TT, i / TT);
                SB();
            }
            asm volatile("" : "+v"(s));  // (the MFMAs of S are not moved behind those of dP)
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                g = mfma32(fv[i], dof[i], g);
                SB();
            }
            // The arithmetic below is written out, and the compiler counts no wait states between an MFMA and
            // such a reader of its result (12 for these on gfx950; s_nop n is n + 1 of them): they are here.  (Without
            // them the first scores were read before they were written where a wavefront had its SIMD to itself.)
            asm volatile("s_nop 11" : "+v"(s), "+v"(g));
            if (__builtin_expect(j >= n_full, 0)) {  // half tile touches the diagonal for this wave
                int li = lane;
                asm volatile("" : "+v"(li));
                const int rel = p0 + wrow0 + (li & 31) - 32 * j - 4 * (li >> 5);  // my_pos - 32j - 4h
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const bool late = 8 * (v >> 2) + (v & 3) > rel;
                    s[v] = late ? -INFINITY : s[v];
                    g[v] = late ? 0.0f : g[v];
                }
            }
            uint32_t pw[8];
            float e[16];
#pragma unroll
            for (int v = 0; v < 16; v += 2) ds_exp2(s[v], s[v + 1], cs, lse2, e[v], e[v + 1]);
#pragma unroll
            for (int v = 0; v < 16; v += 2) pw[v >> 1] = ds_mul_pack(e[v], e[v + 1], g[v], g[v + 1]);
            const bf16x8 ds0 = as_bf16x8(make_uint4(pw[0], pw[1], pw[2], pw[3]));
            const bf16x8 ds1 = as_bf16x8(make_uint4(pw[4], pw[5], pw[6], pw[7]));
            SB();
#pragma unroll
            for (int y = 0; y < 2 * TT; ++y) {
                acc[y % TT] = mfma32(ct[y], y < TT ? ds0 : ds1, acc[y % TT]);
                SB();
            }
        };
#pragma unroll 1
        for (int t = 0; t < n_tiles; ++t) {
            if (t > 0 && (SMALL ? t + 1 < n_tiles : (t & 1) == 0 && t + 2 < n_tiles)) fetch(t);
            if (t == n_tiles - 1) feed.ask();
            const unsigned char *tk = lds_k[t & (KSL - 1)], *tv = lds_v[t & (VSL - 1)];
            if (2 * t <= L) half(2 * t, tk, tv);
            if (2 * t + 1 <= L) half(2 * t + 1, tk + HALF, tv + HALF);
            if (SMALL || (t & 1)) {
                wait_vmem();
                __syncthreads();
                if (ONE && t == 1 && !last_items) count_ready();
            }
        }
        if (ONE && n_tiles == 1 && !last_items) {
            wait_vmem();
            __syncthreads();
            count_ready();
        }
    } else {
    f32x16 sx, sy, gx, gy;  // S and dP - D of the current / next half tile, ping-pong
#pragma unroll
    for (int v = 0; v < 16; ++v) { sx[v] = 0.0f; sy[v] = 0.0f; gx[v] = 0.0f; gy[v] = 0.0f; }

    // Period t: steps 2t-1 and 2t, i.e. A of both halves of tile t (K and V rows), B of
    // the second half of K tile t-1 and of the first half of K tile t.  K tile t sits in
    // slot t mod KSL, V tile t in slot t mod VSL.  Large shape: an even period starts by
    // fetching the tiles of the next two periods into slots that the periods before the
    // last barrier have left; an odd period ends with the wait for them and the barrier.
    // Small shape: every period fetches the next tile (into the slot of K tile t-2, whose
    // second half period t-1 was the last to read, and of V tile t-1) and ends with the
    // wait and the barrier.
    auto period_begin = [&](int t) __attribute__((always_inline)) {
        if (t == 0) return;  // period 0's group went out at start-up
        if (SMALL) {
            if (t + 1 < n_tiles) fetch(t);
        } else {
            if ((t & 1) == 0 && t + 2 < n_tiles) fetch(t);
        }
    };
    auto period_end = [&](int t) __attribute__((always_inline)) {
        if (SMALL || (t & 1)) {
            wait_vmem();      // my share of the tiles of the next period(s) has landed
            __syncthreads();  // ... and everyone's; everyone is done with the tiles they replace
            if (ONE && t == 1 && !last_items) count_ready();  // (every item has a period 1)
        }
        kslot = kslot == KSL - 1 ? 0 : kslot + 1;
    };
    // periods whose two steps are fully inside the wave's unmasked range
    const int t_steady_end = min((L - 1) / 2, (n_full - 1) / 2);  // last t with 2t+1 <= L and 2t < n_full
    auto plain_period = [&](int t) __attribute__((always_inline)) {
        period_begin(t);
        const unsigned char *tk = lds_k[kslot], *tv = lds_v[t & (VSL - 1)];
        const unsigned char *tkp = lds_k[kslot == 0 ? KSL - 1 : kslot - 1] + HALF;  // second half of K tile t-1
#pragma unroll 1
        for (int hh = 0; hh < 2; ++hh) {
            generic(2 * t - 1 + hh, tk + hh * HALF, tv + hh * HALF, hh ? tk : tkp, sx, gx, sy, gy);
            sx = sy;
            gx = gy;
        }
        period_end(t);
    };
    plain_period(0);
    int t = 1;
    for (; t <= t_steady_end; ++t) {
        period_begin(t);
        const unsigned char *tk = lds_k[kslot], *tv = lds_v[t & (VSL - 1)];
        const unsigned char *tkp = lds_k[kslot == 0 ? KSL - 1 : kslot - 1] + HALF;
        bf16x8 fr[4];  // operand fragments in flight
        steady(std::true_type{}, tk, tv, tkp, tk + HALF, tv + HALF, sx, gx, sy, gy, fr);
        steady(std::false_type{}, tk + HALF, tv + HALF, tk, tk, tv, sy, gy, sx, gx, fr);
        period_end(t);
    }
    feed.ask();
#pragma unroll 1
    for (; t <= n_tiles; ++t) plain_period(t);

    }
    feed.post();
    // Nobody reads a tile any more: the staging regions are free.  (The next item needs no barrier
    // of its own before its first tiles: they go to slots that stage nothing.)
    __syncthreads();
    const kernarg_t<BwdParams> out = kernarg<BwdParams>();
    const int next = feed.take();
    // derived after the loop from opaque copies, so that no part of the
    // output addresses is kept in registers during the loop
    int li = lane;
    asm volatile("" : "+v"(li));
    const int on = li & 31, oh = li >> 5, oi = wrow0 + on;
    Stage st;
    st.init(li);
    if (wave_active) st.put_acc(stage, acc, out->scale, on, oh);
    RowBlocks rb_next{};
    if (next >= 0) rb_next = row_blocks<ONE ? 0 : NWQ>(out, out->fwd_items, next);  // (its loads are under way during the stores)
    if (wave_active) {
        st.store(stage, out->dq + ((size_t)qrow0 * out->Hq + head) * D, (uint32_t)out->Hq * D * 2, wrow0, rows);
        if (!ONE && oh == 0 && oi < rows) {
            out->delta[(size_t)head * out->total_q + qrow0 + oi] = nd;
            out->lse2[(size_t)head * out->total_q + qrow0 + oi] = lse2;
        }
    }
    trace_end(out->trace_dq, trace_t0, bid);
    rb = uniform(rb_next);
    return next;
}

// Does dQ work items until none is left.
template <int D, int NWQ, bool PIPED, bool ONE>
__device__ __forceinline__ void dq_loop(DqFeed &feed, unsigned char *lds)
{
    constexpr int NW = ONE ? 0 : NWQ;
    int w = feed.first(feed.begin());
    RowBlocks rb = row_blocks<NW>(kernarg<BwdParams>(), kernarg<BwdParams>()->fwd_items, max(w, 0));
    while (w >= 0) {
        if (rb.has(0)) {
            w = dq_work<D, NWQ, PIPED, ONE>(w, rb, feed, lds);
            if (w == kQueueEmpty) {
                w = feed.other();
                rb = row_blocks<NW>(kernarg<BwdParams>(), kernarg<BwdParams>()->fwd_items, max(w, 0));
            }
        } else {  // the item is too short for this part (the whole workgroup agrees)
            if (ONE && threadIdx.x == 0) count_one(kernarg<BwdParams>()->rows_ready);
            w = feed.again();
            rb = row_blocks<NW>(kernarg<BwdParams>(), kernarg<BwdParams>()->fwd_items, max(w, 0));
        }
    }
}

template <int D, int NWQ, bool PIPED = NWQ == NWQ_LARGE>
__global__ __launch_bounds__(64 * NWQ, PIPED ? 2 : 3) void dq_kernel(const BwdParams prm)
{
    __shared__ __align__(16) unsigned char lds[DqLds<D, NWQ, PIPED>::BYTES];
    __shared__ int work_slot[2];
    if (prm.clear && blockIdx.x == 0) clear_state(prm.clear, SKRULL_BWD_STATE_INTS);
    DqFeed feed{{}, 0, 0, work_slot};
    dq_loop<D, NWQ, PIPED, false>(feed, lds);
}

// ---------------------------------------------------------------------------
// dK / dV, paired waves.
//
// One wave owning 32 key rows would need K, V, dK and dV of those rows in
// registers (192 of them at d=128), which pins it to one wave per SIMD with
// nothing to hide LDS latency or softmax arithmetic behind.  Here two waves
// share the 32 key rows instead:
//   role 0 ("S wave"):  S = Q K^T, P = exp2(S*c - LSE'), dV^T += dO^T P;  holds K, dV
//   role 1 ("dP wave"): dP = dO V^T, dS = P (dP - D), dK^T += Q^T dS;     holds V, dK
// P goes from the first to the second through LDS in MFMA operand format (bf16,
// 4 KB per 64x32 tile).  The unit of work is a tile of 64 query rows; the dP
// wave finishes a tile (dS, dK) one round after the S wave produced its P, so
// one workgroup barrier per round is all the synchronisation there is, and in
// every round both waves of a pair have 32 MFMAs of their own.
// Query tiles (Q, dO, LSE', D) sit in a ring of three LDS slots: a round reads
// the current slot (both waves) and the previous one (dP wave) while the
// asynchronous fetch of the next tile fills the third.
// ---------------------------------------------------------------------------
// Vector-ALU pieces of the dK/dV kernel, written out so that they stay where the
// kernel puts them: between the MFMAs of the next block (plain arithmetic would be
// moved to its first use, behind all of them, and a wave that issues nothing but
// vector instructions for a long stretch slows the MFMAs of the wave it shares a
// SIMD with).
// Four scores -> four probabilities exp2(s * c - l), packed twice: to two bf16 pairs (w0, w1:
// the S wave's own MFMA operand) and to two fp16 pairs (h0, h1: what the dP wave gets).  The
// dP wave only multiplies P element by element, and a mixed-precision multiply takes an fp16
// operand as it is, where a bf16 one costs an instruction to widen first: the extra packing
// here is on the wave of the pair that waits at the barrier, the widening was on the one that
// does not.  (Probabilities are at most 1; fp16 keeps three bits more of them than bf16 and
// goes to zero below 6e-8.)  Every exponential has an instruction between it and the first use
// of its result.
__device__ __forceinline__ void p_quad(const float (&sv)[4], float c, const float4 &l, uint32_t &w0, uint32_t &w1,
                                       uint32_t &h0, uint32_t &h1)
{
    float t0, t1, t2, t3;
    asm volatile("v_fma_f32 %0, %8, %12, -%13\n\t"
                 "v_fma_f32 %1, %9, %12, -%14\n\t"
                 "v_fma_f32 %2, %10, %12, -%15\n\t"
                 "v_fma_f32 %3, %11, %12, -%16\n\t"
                 "v_exp_f32 %0, %0\n\t"
                 "v_exp_f32 %1, %1\n\t"
                 "v_exp_f32 %2, %2\n\t"
                 "v_exp_f32 %3, %3\n\t"
                 "v_cvt_pk_bf16_f32 %4, %0, %1\n\t"
                 "v_cvt_pk_bf16_f32 %5, %2, %3\n\t"
                 "v_cvt_pk_f16_f32 %6, %0, %1\n\t"
                 "v_cvt_pk_f16_f32 %7, %2, %3"
                 : "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3), "=&v"(w0), "=&v"(w1), "=&v"(h0), "=&v"(h1)
                 : "v"(sv[0]), "v"(sv[1]), "v"(sv[2]), "v"(sv[3]), "s"(c), "v"(l.x), "v"(l.y), "v"(l.z), "v"(l.w));
}
// Two packed fp16 P pairs times four (dP - D) values -> two packed bf16 dS pairs.
__device__ __forceinline__ void ds_quad(uint32_t p01, uint32_t p23, const float (&g)[4], uint32_t &w0, uint32_t &w1)
{
    float t0, t1, t2, t3;
    asm volatile("v_fma_mix_f32 %0, %6, %8, 0 op_sel:[0,0,0] op_sel_hi:[1,0,0]\n\t"
                 "v_fma_mix_f32 %1, %6, %9, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]\n\t"
                 "v_fma_mix_f32 %2, %7, %10, 0 op_sel:[0,0,0] op_sel_hi:[1,0,0]\n\t"
                 "v_fma_mix_f32 %3, %7, %11, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]\n\t"
                 "v_cvt_pk_bf16_f32 %4, %0, %1\n\t"
                 "v_cvt_pk_bf16_f32 %5, %2, %3"
                 : "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3), "=&v"(w0), "=&v"(w1)
                 : "v"(p01), "v"(p23), "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]));
}

// PAIRS wave pairs per workgroup: 4 (8 wavefronts, 128 key rows, two wavefronts per SIMD), or,
// at head_dim 64 where 157 registers and 106 KB of LDS allow it, 6 (12 wavefronts, 192 key
// rows, three per SIMD): more wavefronts to overlap with and a third fewer fetches of each
// query tile.  The 12-wavefront shape serves work items of block_n = 192.
constexpr int PAIRS_8W = 4, PAIRS_12W = 6;

// One work item: SUB key rows of one KV head, or what is left of them, and which part of the walk
// over the query heads and tiles that see them.
struct KeyBlock {
    int c, part, parts;            // KV head; part of the work, and of how many
    int shared;                    // 0, or 1 + which counter counts this work item: it stands for a part of a shared item
    int head_lo, g;                // the query heads this part walks over
    int piece, pieces;             // which piece of that walk, and of how many
    int kv0, item_rows;            // first key position; key rows from there on that belong to the item
    int part_row;                  // first row of the pass in a part's partial sums
    int qb, ql, kvl, kbase, qbase; // the (late) segment: position of its first query, rows, keys, packed rows
    int qb_e, ql_e, qbase_e;       // the early chunk that shares the prefix and sees the block (ql_e = 0: none)
};
template <typename P>
__device__ __forceinline__ KeyBlock key_block(const P prm, int SUB, int bid)
{
    KeyBlock r;
    const int BN = prm->keys.BN, Hkv = prm->keys.Hkv, passes = prm->keys.passes, n_split = prm->keys.n_split;
    const int whole = Hkv * passes;
    const int4 *units = prm->keys.units;
    int seq, block, item, sub;
    if (units) {
        const int unit = __builtin_amdgcn_readfirstlane(quotient(bid, prm->keys.inv_whole));
        const i32x4 u = plan_value((const i32x4 *)units, unit);
        const int x = bid - unit * whole;
        r.c = quotient(x, prm->keys.inv_passes);
        sub = x - r.c * passes;
        seq = u.x;
        block = u.y;
        item = u.z & ((1 << SKRULL_UNIT_SHIFT) - 1);
        r.part = u.z >> SKRULL_UNIT_SHIFT;
        r.parts = u.w;
        r.shared = item < n_split ? 1 + item * Hkv + r.c : 0;
    } else {
        const int first = prm->keys.n_whole_first * whole, split = n_split * prm->keys.parts * whole;
        const bool is_split = bid >= first && bid < first + split;
        const int per_item = is_split ? whole * prm->keys.parts : whole;
        const int rel = bid < first ? bid : (is_split ? bid - first : bid - split);
        const int at = __builtin_amdgcn_readfirstlane(rel / per_item), x = rel - at * per_item;
        item = is_split ? at : at + n_split;
        const int y = quotient(x, prm->keys.inv_passes);
        sub = x - y * passes;
        r.part = quotient(y, prm->keys.inv_hkv);
        r.c = y - r.part * Hkv;
        const i32x4 it = plan_value((const i32x4 *)prm->dkv_items, item);
        seq = it.x;
        block = it.y;
        r.parts = 1;
        r.shared = is_split ? 1 + item * Hkv + r.c : 0;
        if (is_split) {
            const int chain = prm->keys.chain;
            r.parts = chain == 0 ? prm->keys.parts
                                 : min(prm->keys.parts, __builtin_amdgcn_readfirstlane((it.w * prm->keys.g + chain - 1) / max(chain, 1)));
        }
    }
    const int prev = max(seq - 1, 0);
    const int shares = plan_value(prm->shares_kv, seq), kvl_e = plan_value(prm->kv_len, prev);
    r.qb = plan_value(prm->q_begin, seq);
    r.ql = plan_value(prm->q_len, seq);
    r.kvl = plan_value(prm->kv_len, seq);
    r.kbase = plan_value(prm->cu_k, seq);
    r.qbase = plan_value(prm->cu_q, seq);
    r.qb_e = plan_value(prm->q_begin, prev);
    r.qbase_e = plan_value(prm->cu_q, prev);
    r.ql_e = plan_value(prm->q_len, prev);
    // A part takes an equal share of the heads where there is one (the parts of neighbouring key
    // blocks then walk the same query tiles at the same time), else an equal piece of the walk over
    // all of them.
    const int g = prm->keys.g, share = __builtin_amdgcn_readfirstlane(g / r.parts);
    const bool by_heads = share * r.parts == g;
    r.g = by_heads ? share : g;
    r.head_lo = r.c * g + (by_heads ? r.part * share : 0);
    r.piece = by_heads ? 0 : r.part;
    r.pieces = by_heads ? 1 : r.parts;
    r.kv0 = block * BN + sub * SUB;
    r.item_rows = r.part < r.parts ? min(BN, r.kvl - block * BN) - sub * SUB : 0;
    r.part_row = prm->keys.part_rows ? item * BN + sub * SUB : r.kbase + r.kv0;
    if (!shares || r.kv0 >= kvl_e) r.ql_e = 0;
    return r;
}

// Counts a part of a shared item (KeyBlock::shared) as stored.
__device__ __forceinline__ void count_part(int shared)
{
    const kernarg_t<BwdParams> prm = kernarg<BwdParams>();
    count_one(prm->parts_stored + (prm->n_parts ? 0 : shared - 1));
}

template <int D, int PAIRS>
struct DkvLds {
    static constexpr int SLOT = 2 * TileGeom<D>::BYTES + 2 * TILE_ROWS * 4;  // Q rows | dO rows | LSE*log2e | D
    static constexpr int RING = 3 * SLOT, P = PAIRS * 2 * 4 * 1024;          // P: exchange [pair][round parity][16-row block][lane*16]
};

// Does work item `bid`, whose keys are `kb`; returns the next one and leaves its keys in `kb`.
// ONE: in one launch with dQ.  `rows_seen`: this workgroup has waited for the rows of dQ's items.  `part_owed`: the part of a shared item
// (KeyBlock::shared) that it did last, stored but not counted yet, or 0; on return this item's.
template <int D, int PAIRS, bool ONE>
__device__ __forceinline__ int dkv_work(const int bid, KeyBlock &kb, DkvFeed &feed, unsigned char *ring, unsigned char *exchange, bool &rows_seen, int &part_owed)
{
    const kernarg_t<BwdParams> prm = kernarg<BwdParams>();
    constexpr int NWP = 2 * PAIRS;   // wavefronts: PAIRS S waves, then PAIRS dP waves
    constexpr int SUB = 32 * PAIRS;  // key rows per workgroup
    constexpr int KS = D / 16, TT = D / 32, QT = TILE_ROWS;
    constexpr int TB = TileGeom<D>::BYTES;
    typedef DkvLds<D, PAIRS> Lds;
    constexpr int SLOT = Lds::SLOT;
    unsigned char (*lds_ring)[SLOT] = (unsigned char (*)[SLOT])ring;
    unsigned char (*lds_p)[2][4][1024] = (unsigned char (*)[2][4][1024])exchange;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int role = wave / PAIRS, pw = wave % PAIRS;  // waves w and w+PAIRS share 32 key rows
    const int n = lane & 31, h = lane >> 5;
    const int c = kb.c, g = kb.g, head_lo = kb.head_lo;
    FragAddr<D> fa;
    fa.init(lane);
    RingLoader<D, NWP> ld;
    ld.init(lane, wave, (uint32_t)prm->Hq * D * 2);
    const uint32_t ring0 = lds_addr(&lds_ring[0][0]);

    const int qb = kb.qb, ql = kb.ql, kvl = kb.kvl, kbase = kb.kbase, qbase = kb.qbase;
    const float cs = prm->scale_log2;
    const uint64_t trace_t0 = trace_begin(prm->trace_dkv);
    const int kv0 = kb.kv0;  // first key position of the pass
    const int krows = min(SUB, kb.item_rows);
    const int wj0 = kv0 + 32 * pw;              // this pair's first key position
    const bool wave_active = 32 * pw < krows;
    const int my_j = wj0 + n;                   // this lane's key position

    // this wave's staging region: ring slots 1 and 2 hold no tile at the start and the end of a
    // pass (eight regions); the waves beyond the eighth use the P exchange area
    typedef WaveStage<D> Stage;
    static_assert(8 * Stage::BYTES <= 2 * SLOT && (NWP - 8) * Stage::BYTES <= Lds::P,
                  "staging regions do not fit the idle part of the LDS");
    const uint32_t stage = wave < 8 ? ring0 + SLOT + (uint32_t)wave * Stage::BYTES
                                    : lds_addr(&lds_p[0][0][0][0]) + (uint32_t)(wave - 8) * Stage::BYTES;
    // B operand held for the whole pass: this lane's key row of K (role 0) or V (role 1).
    bf16x8 bf[KS];
    {
        Stage st;
        st.init(lane);
        u32x4 vk[Stage::N];
        st.load(vk, (role == 0 ? prm->k : prm->v) + ((size_t)kbase * prm->Hkv + c) * D, (uint32_t)prm->Hkv * D * 2, wj0, kvl);
        st.put(stage, vk);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) bf[ks] = fa.rows_at(stage, ks);
    }

    // Query tiles that can see key kv0, numbered 0 .. n_qt-1 in position order: those of
    // the early chunk (segment seq-1, when this prefix is shared by two chunks and the
    // pass starts inside the early chunk's own prefix) and then those of segment seq.
    const int i_first = (max(0, kv0 - qb) / QT) * QT;
    const int n_qt_own = (ql - i_first + QT - 1) / QT;
    const int qb_e = kb.qb_e, ql_e = kb.ql_e, qbase_e = kb.qbase_e;
    const int i_first_e = (max(0, kv0 - qb_e) / QT) * QT;
    const int n_qt_e = ql_e > 0 ? (ql_e - i_first_e + QT - 1) / QT : 0;
    const int n_qt = n_qt_e + n_qt_own;
    // (head, query tile) pairs of the walk described below: this part takes n_iter of them from r0 on
    const bool all = kb.pieces == 1;
    const int r0 = all ? 0 : __builtin_amdgcn_readfirstlane(kb.piece * (n_qt * g) / kb.pieces);
    const int n_iter = (all ? n_qt * g : __builtin_amdgcn_readfirstlane((kb.piece + 1) * (n_qt * g) / kb.pieces)) - r0;
    const int first_up = r0 == 0 ? 0 : __builtin_amdgcn_readfirstlane(r0 / g);
    const int head0 = r0 - first_up * g, tile0 = n_qt - 1 - first_up;
    // tile t -> first global position of its segment, rows of the segment, first row of the tile
    auto tile_qb = [&](int t) __attribute__((always_inline)) { return t < n_qt_e ? qb_e : qb; };
    auto tile_ql = [&](int t) __attribute__((always_inline)) { return t < n_qt_e ? ql_e : ql; };
    auto tile_i0 = [&](int t) __attribute__((always_inline)) {
        return t < n_qt_e ? i_first_e + t * QT : i_first + (t - n_qt_e) * QT;
    };

    f32x16 acc[TT];  // dV^T (role 0) or dK^T (role 1) of this lane's key
    zero_acc(acc);

    // wave 2 fetches a tile's LSE', wave 3 its -D (both kept from here on: read again in every
    // round, the pointers cost these two waves the latency of a scalar load per round)
    const bool row_scalars = wave == 2 || wave == 3;
    const float *scalars = wave == 2 ? prm->lse2 : prm->delta;
    const int scalars_at = 2 * TB + (wave == 2 ? 0 : QT * 4);
    int total_q = prm->total_q;
    asm volatile("" : "+s"(scalars), "+s"(total_q));
    // fetch of tile (head th of the group, query tile tq_idx) into ring slot `slot`
    auto fetch = [&](int th, int tq_idx, int slot) __attribute__((always_inline)) {
        const int head = head_lo + th;
        const int i0 = tile_i0(tq_idx);
        const int rows = tile_ql(tq_idx);
        const int first_row = tq_idx < n_qt_e ? qbase_e : qbase;
        const uint32_t base = ring0 + (uint32_t)slot * SLOT;
        const size_t hoff = ((size_t)first_row * prm->Hq + head) * D;
        // rows past the end of the segment read as zero (and are masked)
        ld.load(ld.rsrc(prm->q + hoff, rows), base, i0, wave);
        ld.load(ld.rsrc(prm->d_o + hoff, rows), base + TB, i0, wave);
        if (row_scalars) {
            const i32x4 r = rsrc_words(scalars + (size_t)head * total_q + first_row, (uint32_t)rows * 4);
            if (ONE) dma_b32_shared(r, base + scalars_at, lane * 4, i0 * 4);
            else dma_b32(r, base + scalars_at, lane * 4, i0 * 4);
        }
    };

    if (ONE && !rows_seen) {  // this workgroup's first item
        const kernarg_t<BwdParams> wait = kernarg<BwdParams>();
        if (tid == 0)
            while (__hip_atomic_load(wait->rows_ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < wait->n_work_dq) __builtin_amdgcn_s_sleep(4);
        __syncthreads();  // (-D and LSE are read past the L2: with a fence by each workgroup, which empties it, dK/dV began 30 us later)
        rows_seen = true;
    }
    fetch(head0, tile0, 0);
    wait_vmem();
    __syncthreads();
    if (ONE && part_owed && tid == 0) count_part(part_owed);  // (everyone's stores of the item before are done)

    // Round T: ring slot T % 3 holds (head t % g, query tile n_qt - 1 - t / g), t = r0 + T: heads
    // innermost, query tiles from the end of the sequence down to the block's
    // diagonal.  Every workgroup of a sequence then starts at the same tile and the
    // ones running together walk the same tiles at the same time, which is what
    // lets the XCD's L2 serve most of their fetches.
    // A pair's LIVE rounds are a prefix of the sequence: the tiles whose last query still
    // precedes the pair's first key are the lowest ones, walked last.  Each role runs its
    // live rounds in ONE loop with ONE sequence of MFMAs (masks, where a tile needs them,
    // only change scores before the exponentials), then idles through the rest with the
    // fetches and barriers every wave must take part in.  With alternative MFMA paths
    // inside one loop the compiler reconciled their register assignments with ~100
    // register copies per round.
    auto tile_live = [&](int t) __attribute__((always_inline)) {
        return tile_qb(t) + tile_i0(t) + QT - 1 >= wj0;
    };
    int n_live = 0;  // live rounds of this pair
    if (wave_active) {
        int dead_tiles = 0;
        if (n_qt_e > 0) {  // the early chunk's lowest tile may be dead; the late chunk's never is
            if (!tile_live(0)) dead_tiles = 1;
        } else {
            while (dead_tiles < n_qt && !tile_live(dead_tiles)) ++dead_tiles;
        }
        n_live = max(0, min(n_iter, (n_qt - dead_tiles) * g - r0));
    }
    int nh = head0 + 1, nq = tile0, cq = tile0, slot = 0;  // cq: tile of this round; (nh, nq): head, tile of the next
    if (nh == g) { nh = 0; --nq; }
    // start of a round: fetch the next round's tile; end: wait, barrier, advance
    auto round_begin = [&](int T) __attribute__((always_inline)) {
        if (T + 1 < n_iter) fetch(nh, nq, slot == 2 ? 0 : slot + 1);
    };
    auto round_end = [&]() __attribute__((always_inline)) {
        wait_vmem();      // my share of the next tile has landed
        __syncthreads();  // ... and everyone's; P of this round is visible; the previous slot is free
        slot = slot == 2 ? 0 : slot + 1;
        cq = nq;
        if (++nh == g) { nh = 0; --nq; }
    };
    int T = 0;
    if (role == 0) {
#pragma unroll 1
        for (; T < n_live; ++T) {
            round_begin(T);
            const unsigned char *cur = lds_ring[slot];
            const int i0 = tile_i0(cq);  // first query row of the tile inside its segment
            const int qb_t = tile_qb(cq), ql_t = tile_ql(cq);
            const unsigned char *tq = cur, *tdo = cur + TB;
            const float *t_lse = (const float *)(cur + 2 * TB);
            unsigned char *px = lds_p[pw][T & 1][0];
            // masked pairs: key past the query (causal) or query row past the end
            const bool need_mask = (qb_t + i0 < wj0 + 31) || (i0 + QT > ql_t);
            // scores of masked pairs become -inf (probability 0) before the exponentials
            auto mask_block = [&](f32x16 &sb, int b) __attribute__((always_inline)) {
                // (the asm also keeps this block behind its branch: turned into selects it
                // would run in every round)
                int li = lane;
                asm volatile("" : "+v"(li));  // thresholds formed here, not kept across rounds
                const int row0 = i0 + 32 * b + 4 * (li >> 5);            // + 8*vb + e = query row
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int i = row0 + 8 * (v >> 2) + (v & 3);
                    sb[v] = (wj0 + (li & 31) > qb_t + i || i >= ql_t) ? -INFINITY : sb[v];
                }
            };
            f32x16 s[2];
            bf16x8 fr[4];
            // S of the first 32 rows; operand reads run three MFMAs ahead
#pragma unroll
            for (int x = 0; x < 3; ++x) fr[x] = fa.rows(tq, 0, x);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if (ks == 0) {
                    f32x16 z;
#pragma unroll
                    for (int v = 0; v < 16; ++v) z[v] = 0.0f;
                    s[0] = mfma32(fr[0], bf[0], z);
                } else {
                    s[0] = mfma32(fr[ks % 4], bf[ks], s[0]);
                }
                const int nx = ks + 3;
                fr[nx % 4] = nx < KS ? fa.rows(tq, 0, nx) : fa.rows(tq, 1, nx - KS);
                SB();
            }
            if (__builtin_expect(need_mask, 0)) mask_block(s[0], 0);
            // S of the second 32 rows with the probabilities of the first behind its
            // MFMAs, then dV of the first with the probabilities of the second
            uint32_t w[2][8];
            uint32_t hw[4];  // fp16 copies of two quads at a time, on their way to the dP wave
            bf16x8 ft[4];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if (ks == 0) {
                    f32x16 z;
#pragma unroll
                    for (int v = 0; v < 16; ++v) z[v] = 0.0f;
                    s[1] = mfma32(fr[(KS + 0) % 4], bf[0], z);
                } else {
                    s[1] = mfma32(fr[(KS + ks) % 4], bf[ks], s[1]);
                }
                const int nx = ks + 3;
                if (nx < KS) fr[(KS + nx) % 4] = fa.rows(tq, 1, nx);
                if (KS == 8 ? (ks % 2 == 1) : true) {
                    const int vb = KS == 8 ? ks / 2 : ks;
                    const float4 l4 = *(const float4 *)(t_lse + 8 * vb + 4 * h);
                    const float sv[4] = {s[0][4 * vb], s[0][4 * vb + 1], s[0][4 * vb + 2], s[0][4 * vb + 3]};
                    p_quad(sv, cs, l4, w[0][2 * vb], w[0][2 * vb + 1], hw[2 * (vb & 1)], hw[2 * (vb & 1) + 1]);
                    if (vb & 1) *(uint4 *)(px + (vb >> 1) * 1024 + lane * 16) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
                }
                if (ks >= KS - 3) ft[(ks - (KS - 3))] = fa.cols(tdo, (ks - (KS - 3)) % TT, (ks - (KS - 3)) / TT);
                SB();
            }
            if (__builtin_expect(need_mask, 0)) mask_block(s[1], 1);
            const bf16x8 pb0 = as_bf16x8(make_uint4(w[0][0], w[0][1], w[0][2], w[0][3]));
            const bf16x8 pb1 = as_bf16x8(make_uint4(w[0][4], w[0][5], w[0][6], w[0][7]));
            // dV of rows 0..31 (2 x TT MFMAs); probabilities of rows 32..63 behind them
#pragma unroll
            for (int m = 0; m < 2 * TT; ++m) {
                acc[m % TT] = mfma32(ft[m % 4], m < TT ? pb0 : pb1, acc[m % TT]);
                const int nx = m + 3;
                ft[nx % 4] = fa.cols(tdo, nx % TT, nx / TT);  // runs on into rows 32..63
                if (TT == 4 ? (m % 2 == 1) : true) {
                    const int vb = TT == 4 ? m / 2 : m;
                    const float4 l4 = *(const float4 *)(t_lse + 32 + 8 * vb + 4 * h);
                    const float sv[4] = {s[1][4 * vb], s[1][4 * vb + 1], s[1][4 * vb + 2], s[1][4 * vb + 3]};
                    p_quad(sv, cs, l4, w[1][2 * vb], w[1][2 * vb + 1], hw[2 * (vb & 1)], hw[2 * (vb & 1) + 1]);
                    if (vb & 1) *(uint4 *)(px + (2 + (vb >> 1)) * 1024 + lane * 16) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
                }
                SB();
            }
            const bf16x8 pb2 = as_bf16x8(make_uint4(w[1][0], w[1][1], w[1][2], w[1][3]));
            const bf16x8 pb3 = as_bf16x8(make_uint4(w[1][4], w[1][5], w[1][6], w[1][7]));
            // dV of rows 32..63
#pragma unroll
            for (int m = 2 * TT; m < 4 * TT; ++m) {
                acc[m % TT] = mfma32(ft[m % 4], m < 3 * TT ? pb2 : pb3, acc[m % TT]);
                const int nx = m + 3;
                if (nx < 4 * TT) ft[nx % 4] = fa.cols(tdo, nx % TT, nx / TT);
                SB();
            }
            round_end();
        }
    } else {
        f32x16 dp[2];  // dP - D of the previous round's tile
        zero_acc(dp);
        // first live round: dP - D of its tile only
        if (n_live > 0) {
            round_begin(T);
            const unsigned char *cur = lds_ring[slot];
            const unsigned char *tdo = cur + TB;
            const float *t_nd = (const float *)(cur + 2 * TB) + QT;  // -D of this round's tile
            // accumulator start of a 32-row block of dP: -D of its rows
            auto neg_d = [&](int b) __attribute__((always_inline)) {
                f32x16 z;
#pragma unroll
                for (int vb = 0; vb < 4; ++vb) {
                    const float4 d4 = *(const float4 *)(t_nd + 32 * b + 8 * vb + 4 * h);
                    z[4 * vb] = d4.x; z[4 * vb + 1] = d4.y; z[4 * vb + 2] = d4.z; z[4 * vb + 3] = d4.w;
                }
                return z;
            };
            {
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    dp[b] = neg_d(b);
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        dp[b] = mfma32(fa.rows(tdo, b, ks), bf[ks], dp[b]);
                        if (ks % 4 == 3) SB();
                    }
                }
            }
            round_end();
            ++T;
        }
#pragma unroll 1
        for (; T < n_live; ++T) {
            round_begin(T);
            const int slot_prev = slot == 0 ? 2 : slot - 1;
            const unsigned char *cur = lds_ring[slot], *prv = lds_ring[slot_prev];
            const unsigned char *tdo = cur + TB;
            const float *t_nd = (const float *)(cur + 2 * TB) + QT;  // -D of this round's tile
            const unsigned char *pp = lds_p[pw][(T - 1) & 1][0];
            // accumulator start of a 32-row block of dP: -D of its rows
            auto neg_d = [&](int b) __attribute__((always_inline)) {
                f32x16 z;
#pragma unroll
                for (int vb = 0; vb < 4; ++vb) {
                    const float4 d4 = *(const float4 *)(t_nd + 32 * b + 8 * vb + 4 * h);
                    z[4 * vb] = d4.x; z[4 * vb + 1] = d4.y; z[4 * vb + 2] = d4.z; z[4 * vb + 3] = d4.w;
                }
                return z;
            };
            // dS of 16 rows (block b, half kb) of the previous tile from its P and dP - D
            auto ds_half = [&](const uint4 &p4, const f32x16 &g, int kb, uint32_t (&w)[4]) __attribute__((always_inline)) {
                const float g0[4] = {g[8 * kb], g[8 * kb + 1], g[8 * kb + 2], g[8 * kb + 3]};
                const float g1[4] = {g[8 * kb + 4], g[8 * kb + 5], g[8 * kb + 6], g[8 * kb + 7]};
                ds_quad(p4.x, p4.y, g0, w[0], w[1]);
                ds_quad(p4.z, p4.w, g1, w[2], w[3]);
            };
            // Both tiles live: dP of this tile's first 32 rows with dS of the previous
            // tile's first 32 rows behind its MFMAs; dK of those rows with the second dS
            // behind; then dK of the second rows and dP of this tile's second rows.
            f32x16 dpn;
            bf16x8 fr[4], ft[4];
            uint32_t w[4][4];
            // what the first MFMA waits for is asked for first (when the barrier opens all eight
            // waves queue their reads at once): -D, the start of its accumulator, and dO
            dpn = neg_d(0);
#pragma unroll
            for (int x = 0; x < 3; ++x) fr[x] = fa.rows(tdo, 0, x);
            SB();
            const uint4 p0 = *(const uint4 *)(pp + 0 * 1024 + lane * 16);
            const uint4 p1 = *(const uint4 *)(pp + 1 * 1024 + lane * 16);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                dpn = mfma32(fr[ks % 4], bf[ks], dpn);
                const int nx = ks + 3;
                if (nx < KS) fr[nx % 4] = fa.rows(tdo, 0, nx);
                if (ks == (KS == 8 ? 1 : 0)) ds_half(p0, dp[0], 0, w[0]);
                if (ks == (KS == 8 ? 4 : 2)) ds_half(p1, dp[0], 1, w[1]);
                if (ks >= KS - 3) ft[ks - (KS - 3)] = fa.cols(prv, (ks - (KS - 3)) % TT, (ks - (KS - 3)) / TT);
                SB();
            }
            const uint4 p2 = *(const uint4 *)(pp + 2 * 1024 + lane * 16);
            const uint4 p3 = *(const uint4 *)(pp + 3 * 1024 + lane * 16);
            const bf16x8 db0 = as_bf16x8(make_uint4(w[0][0], w[0][1], w[0][2], w[0][3]));
            const bf16x8 db1 = as_bf16x8(make_uint4(w[1][0], w[1][1], w[1][2], w[1][3]));
#pragma unroll
            for (int m = 0; m < 2 * TT; ++m) {
                acc[m % TT] = mfma32(ft[m % 4], m < TT ? db0 : db1, acc[m % TT]);
                const int nx = m + 3;
                ft[nx % 4] = fa.cols(prv, nx % TT, nx / TT);  // runs on into rows 32..63
                if (m == (TT == 4 ? 1 : 0)) ds_half(p2, dp[1], 0, w[2]);
                if (m == (TT == 4 ? 4 : 2)) ds_half(p3, dp[1], 1, w[3]);
                SB();
            }
            const bf16x8 db2 = as_bf16x8(make_uint4(w[2][0], w[2][1], w[2][2], w[2][3]));
            const bf16x8 db3 = as_bf16x8(make_uint4(w[3][0], w[3][1], w[3][2], w[3][3]));
            // dS of the previous tile is complete: its dP - D registers take the start of this
            // tile's second block (-D) now, eight MFMAs before the products that need it
            dp[1] = neg_d(1);
#pragma unroll
            for (int x = 0; x < 3; ++x) fr[x] = fa.rows(tdo, 1, x);
            SB();
#pragma unroll
            for (int m = 2 * TT; m < 4 * TT; ++m) {
                acc[m % TT] = mfma32(ft[m % 4], m < 3 * TT ? db2 : db3, acc[m % TT]);
                const int nx = m + 3;
                if (nx < 4 * TT) ft[nx % 4] = fa.cols(prv, nx % TT, nx / TT);
                SB();
            }
            dp[0] = dpn;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                dp[1] = mfma32(fr[ks % 4], bf[ks], dp[1]);
                const int nx = ks + 3;
                if (nx < KS) fr[nx % 4] = fa.rows(tdo, 1, nx);
                SB();
            }
            round_end();
        }
        // the round after the last live one: dS and dK of the last live tile
        if (n_live > 0) {
            round_begin(T);
            const int slot_prev = slot == 0 ? 2 : slot - 1;
            const unsigned char *prv = lds_ring[slot_prev];
            const unsigned char *pp = lds_p[pw][(T - 1) & 1][0];
            // dS of 16 rows (block b, half kb) of the previous tile from its P and dP - D
            auto ds_half = [&](const uint4 &p4, const f32x16 &g, int kb, uint32_t (&w)[4]) __attribute__((always_inline)) {
                const float g0[4] = {g[8 * kb], g[8 * kb + 1], g[8 * kb + 2], g[8 * kb + 3]};
                const float g1[4] = {g[8 * kb + 4], g[8 * kb + 5], g[8 * kb + 6], g[8 * kb + 7]};
                ds_quad(p4.x, p4.y, g0, w[0], w[1]);
                ds_quad(p4.z, p4.w, g1, w[2], w[3]);
            };
            {
#pragma unroll
                for (int kbg = 0; kbg < 4; ++kbg) {
                    const uint4 p4 = *(const uint4 *)(pp + kbg * 1024 + lane * 16);
                    uint32_t w[4];
                    ds_half(p4, dp[kbg >> 1], kbg & 1, w);
                    const bf16x8 db = as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
#pragma unroll
                    for (int tt = 0; tt < TT; ++tt) acc[tt] = mfma32(fa.cols(prv, tt, kbg), db, acc[tt]);
                    SB();
                }
            }
            round_end();
            ++T;
        }
    }
    // rounds without work for this pair: keep fetching and meeting the others
    feed.ask();
#pragma unroll 1
    for (; T <= n_iter; ++T) {
        round_begin(T);
        if (T == n_iter) feed.post();
        round_end();
    }
    // (the last round ended with a barrier: nobody reads a tile or P any more; the next item's
    // first tile goes to slot 0, where nothing is staged)
    const kernarg_t<BwdParams> out = kernarg<BwdParams>();
    const int next = feed.take(), parts = kb.parts, part = kb.part, part_row = kb.part_row;
    KeyBlock kb_next{};
    if (next >= 0) kb_next = key_block(out, SUB, next);  // (its loads are under way during the stores)
    if (wave_active) {
        if (parts == 1) {
            Stage st;
            st.init(lane);
            st.put_acc(stage, acc, role == 0 ? 1.0f : out->scale, n, h);
            st.store(stage, (role == 0 ? out->dv : out->dk) + ((size_t)kbase * out->Hkv + c) * D,
                     (uint32_t)out->Hkv * D * 2, wj0, kvl);
        } else if (my_j < kvl) {
            const size_t rows = out->keys.part_rows ? out->keys.part_rows : out->total_k;
            float *sums = role == 0 ? out->dv_part : out->dk_part;
            if (ONE) {
                const int valid = min(32, kvl - wj0);
                const size_t at = ((size_t)part * out->Hkv + c) * rows + part_row + (wj0 - kv0);
                AccTile<D>::store(shared_buffer(sums + at * D, valid * D * 4), acc, n, h, valid);
            } else {
                const size_t at = (part * rows + part_row + (my_j - kv0)) * out->Hkv + c;
                store_rows_f32<TT>(sums + at * D, acc, h);
            }
        }
    }
    trace_end(out->trace_dkv, trace_t0, bid);
    part_owed = kb.shared;
    kb = uniform(kb_next);
    return next;
}

// Does dK/dV work items until none is left.
template <int D, int PAIRS, bool ONE>
__device__ __forceinline__ void dkv_loop(DkvFeed &feed, unsigned char *ring, unsigned char *exchange)
{
    bool rows_seen = !ONE;
    int part_owed = 0;
    int w = feed.first(feed.begin());
    KeyBlock kb = key_block(kernarg<BwdParams>(), 32 * PAIRS, max(w, 0));
    while (w >= 0) {
        if (kb.item_rows > 0) {
            w = dkv_work<D, PAIRS, ONE>(w, kb, feed, ring, exchange, rows_seen, part_owed);
            if (w == kQueueEmpty) {
                if (ONE && part_owed) {  // (the search takes microseconds)
                    wait_vmem();
                    __syncthreads();
                    if (threadIdx.x == 0) count_part(part_owed);
                    part_owed = 0;
                }
                w = feed.other();
                kb = key_block(kernarg<BwdParams>(), 32 * PAIRS, max(w, 0));
            }
        } else {  // the item has no second pass, or no such part (the whole workgroup agrees)
            if (ONE && kb.shared && threadIdx.x == 0) count_part(kb.shared);
            w = feed.again();
            kb = key_block(kernarg<BwdParams>(), 32 * PAIRS, max(w, 0));
        }
    }
    if (ONE && part_owed) {
        wait_vmem();
        __syncthreads();
        if (threadIdx.x == 0) count_part(part_owed);
    }
}

template <int D, int PAIRS>
__global__ __launch_bounds__(128 * PAIRS, PAIRS == PAIRS_12W ? 3 : 2) void dkv_kernel(const BwdParams prm)
{
    // (two arrays: in one, the compiler took a store to the exchange for one to the ring, and dK/dV of long chains 0.5 % longer)
    __shared__ __align__(16) unsigned char ring[DkvLds<D, PAIRS>::RING], exchange[DkvLds<D, PAIRS>::P];
    __shared__ int work_slot[2];
    DkvFeed feed{{}, 0, 0, work_slot};
    dkv_loop<D, PAIRS, false>(feed, ring, exchange);
}

// Sums of the partial gradients of the items that several workgroups shared, rounded once (the same as
// dkv_reduce_kernel, in the launch that leaves them): a 32-row tile of an item, dK and dV, at a time, handed out
// to workgroups that find no dK/dV item left; a few register quads of the tile (AccTile) to a wavefront, of all parts at once.  The items with the
// longest chains come first, as their parts did, so most pieces wait for nothing.  A wait ends: the parts are all handed out by
// then, to workgroups that wait for nothing before they have counted theirs.
template <int D, int PAIRS>
__device__ __forceinline__ void sums_loop(int *slot)
{
    constexpr int QUADS = AccTile<D>::QUADS, MINE = (2 * QUADS + 2 * PAIRS - 1) / (2 * PAIRS);  // quads of a wavefront
    constexpr int AT_ONCE = kMaxParts;  // parts asked for at once
    const kernarg_t<BwdParams> prm = kernarg<BwdParams>();
    const int Hkv = prm->Hkv, BN = prm->keys.BN, per_item = (BN + 31) / 32;
    const int n_sums = prm->keys.n_split * Hkv * per_item;
    auto claim = [&]() __attribute__((always_inline)) {
        return __hip_atomic_fetch_add(prm->next_sum + opaque(0), opaque(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    int next = 0;
    if (threadIdx.x == 0) next = claim();
    const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t part_rows = prm->keys.part_rows ? prm->keys.part_rows : prm->total_k;
    for (;;) {
        __syncthreads();  // (everyone has read the slot)
        if (threadIdx.x == 0) *slot = next;
        __syncthreads();
        const int w = __builtin_amdgcn_readfirstlane(*slot);
        if (w >= n_sums) break;
        if (threadIdx.x == 0) next = claim();
        const int x = w / per_item, item = x / Hkv, c = x - item * Hkv, row0 = (w - x * per_item) * 32;
        const i32x4 it = plan_value((const i32x4 *)prm->dkv_items, item);
        const int kv0 = it.y * BN;
        const int rows = min(32, min(BN, plan_value(prm->kv_len, it.x) - kv0) - row0);
        const int krow = plan_value(prm->cu_k, it.x) + kv0 + row0;
        const int chain = prm->keys.chain;
        const int parts = chain == 0 ? prm->keys.parts : min(prm->keys.parts, (it.w * prm->keys.g + chain - 1) / chain);
        if (rows <= 0) continue;
        if (threadIdx.x == 0) {
            const int32_t *stored = prm->parts_stored + (prm->n_parts ? 0 : x);
            // (without a list of units every shared item has as many work items as the one of the most parts: those past its own
            // parts are empty, and are counted as soon as somebody takes them, before the parts under way are stored)
            const int all = prm->n_parts ? prm->n_parts : (prm->keys.units ? parts : prm->keys.parts) * prm->keys.passes;
            while (__hip_atomic_load(stored, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < all) __builtin_amdgcn_s_sleep(4);
        }
        __syncthreads();
        const size_t first = c * part_rows + (prm->keys.part_rows ? (size_t)item * BN + row0 : (size_t)krow);
        const size_t step = part_rows * Hkv * D;
        f32x4 a[MINE];
        for (int p0 = 0; p0 < parts; p0 += AT_ONCE) {
            u32x4 b[AT_ONCE][MINE];
#pragma unroll
            for (int k = 0; k < AT_ONCE; ++k)
                if (p0 + k < parts) {
#pragma unroll
                    for (int j = 0; j < MINE; ++j) {
                        const int i = wave * MINE + j;  // (past dV's last quad: reads as zero)
                        const float *sums = (i < QUADS ? prm->dk_part : prm->dv_part) + first * D + (p0 + k) * step;
                        b[k][j] = __builtin_amdgcn_raw_buffer_load_b128(shared_buffer(sums, i < 2 * QUADS ? rows * D * 4 : 0), AccTile<D>::offset(i % QUADS, n, h, rows), 0, kPastL2);
                    }
                }
#pragma unroll
            for (int k = 0; k < AT_ONCE; ++k)
                if (p0 + k < parts) {
#pragma unroll
                    for (int j = 0; j < MINE; ++j) a[j] = p0 + k == 0 ? __builtin_bit_cast(f32x4, b[k][j]) : a[j] + __builtin_bit_cast(f32x4, b[k][j]);
                }
        }
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const int i = wave * MINE + j;
            const float mul = i < QUADS ? prm->scale : 1.0f;
            const float a0 = a[j][0] * mul, a1 = a[j][1] * mul, a2 = a[j][2] * mul, a3 = a[j][3] * mul;
            if (i < 2 * QUADS && n < rows)
                *(uint2 *)((i < QUADS ? prm->dk : prm->dv) + ((size_t)(krow + n) * Hkv + c) * D + 8 * (i % QUADS) + 4 * h) = make_uint2(pack_bf16(a0, a1), pack_bf16(a2, a3));
        }
    }
}

// dQ, then dK/dV, then sums, in one launch: a workgroup that finds no dQ item left goes on with dK/dV items, so that the chip has
// work while the last dQ items end.  These need -D and LSE*log2(e) of rows that other workgroups may still be at, but
// only from their start: a dQ item forms both before its first product, so where every item has been handed out all that is
// needed follows within microseconds.  The wait for it ends: items are only handed out to workgroups that run, and none
// of these waits before it has counted its items as ready.
// As two launches, from a workgroup's last dQ item to the first dK/dV item on its compute unit 14 to 19 us pass (the longest item's
// end, the end of one launch and the start of the next), 2.5 this way.  Then the sums of shared dK/dV items, while the last of the
// other items end; from dK/dV to the next call's dQ over a launch for them 17 us passed.  Backward in three launches, with
// the sums in a second one, and this: 26,624 tokens in 64 sequences, 14/2 heads of 64, 214, 197 and 193 us; 16,384 in 20 232, 215 and 211;
// 13,312 in 10, 28/4 heads of 128, 837, 828 and 822; 32,768 of 16 to 1,024, 32/8 heads of 128, which shares none, 634 and 629; long chains
// the same within 0.5 %; 932 tokens, 4/4 heads of 64, 29 and 22.6.  (With one counter for the parts of all items, which the sums then wait
// for at the end, the sums cost as much as in a launch of their own: 209 us where this takes 196.)  dQ workgroups have as many wavefronts as those of dK/dV here, 8 or 12, and
// leave some without work where the plan's units are smaller.  Launches of many units of 4 stay two: three such workgroups share a
// compute unit there (slices of three long sequences, 14/2 heads of 64: 4.68 ms, in one launch 5.1).
template <int D, int PAIRS>
__global__ __launch_bounds__(128 * PAIRS, PAIRS == PAIRS_12W ? 3 : 2) void bwd_kernel(const BwdParams prm)
{
    constexpr int NW = 2 * PAIRS;
    constexpr bool PIPED = NW == NWQ_LARGE;
    typedef DqLds<D, NW, PIPED> Dq;
    typedef DkvLds<D, PAIRS> Dkv;
    // (dK/dV's two arrays are one where there is no room for them beside each other)
    constexpr int APART = D == 64 ? Dkv::P : 16, TOGETHER = D == 64 ? Dkv::RING : Dkv::RING + Dkv::P;
    __shared__ __align__(16) unsigned char lds[Dq::BYTES > TOGETHER ? Dq::BYTES : TOGETHER], apart[APART];
    __shared__ int work_slot[2];
    if (prm.clear && blockIdx.x == 0) clear_state(prm.clear, SKRULL_BWD_STATE_INTS);
    {
        DqFeed feed{{}, 0, 0, work_slot};
        dq_loop<D, NW, PIPED, true>(feed, lds);
    }
    {
        DkvFeed feed{{}, 0, 0, work_slot};
        dkv_loop<D, PAIRS, true>(feed, lds, D == 64 ? apart : lds + Dkv::RING);
    }
    if (kernarg<BwdParams>()->keys.n_split > 0) sums_loop<D, PAIRS>(work_slot);
}

// Sum of the partial gradients of the items that several workgroups shared, rounded once:
// out = bf16(mul * sum_p part[p]).  Block (x, y, z): KV head x % Hkv of item x / Hkv, 8 or 16 of its rows,
// dK or dV; a thread has one place of four columns.  (With 32 rows to a block it had up to four, summed one
// after another: 900 tokens, 28/4 heads of 128, in seven parts 10.2 us, now 6.2; 1,500: 10.4 and 8.0.)
// Large ones are bound by the partial sums' bytes; only rows that were shared are touched.
template <int D> constexpr int REDUCE_ROWS = 1024 / D;
template <int D>
__global__ __launch_bounds__(256) void dkv_reduce_kernel(const BwdParams prm)
{
    const int item = blockIdx.x / prm.Hkv, c = blockIdx.x - item * prm.Hkv;
    const int4 it = prm.dkv_items[item];
    const int row0 = blockIdx.y * REDUCE_ROWS<D>;
    const int kv0 = it.y * prm.keys.BN;
    const int rows = min(REDUCE_ROWS<D>, min(prm.keys.BN, prm.kv_len[it.x] - kv0) - row0);
    const int krow = prm.cu_k[it.x] + kv0 + row0;
    const int parts = parts_of(prm.keys, it.w);
    const size_t part_rows = prm.keys.part_rows ? prm.keys.part_rows : prm.total_k;
    const size_t prow = prm.keys.part_rows ? (size_t)item * prm.keys.BN + row0 : (size_t)krow;
    const bool dk = blockIdx.z == 0;
    const float4 *part = (const float4 *)(dk ? prm.dk_part : prm.dv_part);
    uint2 *out = (uint2 *)(dk ? prm.dk : prm.dv);
    const float mul = dk ? prm.scale : 1.0f;
    const int r = threadIdx.x / (D / 4), q = threadIdx.x % (D / 4);
    if (r >= rows) return;
    const float4 *src = part + ((prow + r) * prm.Hkv + c) * (D / 4) + q;
    float4 a = *src;
    for (int p = 1; p < parts; ++p) {
        const float4 b = src[(size_t)p * part_rows * prm.Hkv * (D / 4)];
        a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    uint2 w;
    w.x = pack_bf16(a.x * mul, a.y * mul);
    w.y = pack_bf16(a.z * mul, a.w * mul);
    out[((size_t)(krow + r) * prm.Hkv + c) * (D / 4) + q] = w;
}

int dkv_pairs(const skrull_attn_plan_t *p) { return (p->d == 64 && p->BN == 32 * PAIRS_12W) ? PAIRS_12W : PAIRS_8W; }

RowLaunch rows_dq_alone(const skrull_attn_plan_t *p)
{
    if (p->d == 128) return row_launch<dq_kernel<128, NWQ_LARGE>>(p, NWQ_LARGE);
    if (p->dq_waves == NWQ_SMALL && p->dq_piped) return row_launch<dq_kernel<64, NWQ_SMALL, true>>(p, NWQ_SMALL);
    if (p->dq_waves == NWQ_SMALL) return row_launch<dq_kernel<64, NWQ_SMALL>>(p, NWQ_SMALL);
    if (p->dq_waves == NWQ_WIDE) return row_launch<dq_kernel<64, NWQ_WIDE>>(p, NWQ_WIDE);
    return row_launch<dq_kernel<64, NWQ_LARGE>>(p, NWQ_LARGE);
}

// Whether a launch of dK/dV has more work items than the chip holds at once.
bool dkv_queued(const skrull_attn_plan_t *p)
{
    const int n = grid_dkv(p);
    if (p->d == 128) return wants_queue<dkv_kernel<128, PAIRS_8W>>(128 * PAIRS_8W, n);
    return dkv_pairs(p) == PAIRS_12W ? wants_queue<dkv_kernel<64, PAIRS_12W>>(128 * PAIRS_12W, n) : wants_queue<dkv_kernel<64, PAIRS_8W>>(128 * PAIRS_8W, n);
}

// Whether a backward is one launch, of workgroups that take dQ items, then dK/dV items.
template <int D, int PAIRS> bool is_one(const skrull_attn_plan_t *p)
{
    const RowLaunch dq = rows_dq_alone(p);
    if (p->dq_waves == NWQ_SMALL && dq.queued) return false;
    if (D == 64 && PAIRS == PAIRS_8W && p->dq_waves > 8) return false;
    // Where dQ would be a plain grid, and dK/dV too or its items short, separate launches look into no queues, which costs
    // each workgroup of the one launch an atomic or more on few lines; what it saves are gaps and, the longer the items, the wait for the last of dQ.
    // Of 581 such backwards, 21 to 5,600 tokens, all kinds of heads: 277 in one launch 14 % less time than as separate ones (6 % more to 35 % less), 304 separately
    // 5 % less than in one (28 % more to 36 % less; against a launch for each of dQ, dK/dV and sums, queues cleared by one before them, all
    // 8 % less and 5 % more at worst, in one launch throughout 58 % more at worst).
    if (!dq.queued && (!dkv_queued(p) || p->longest_seq <= 160) && dq.n_work + grid_dkv(p) > 80 + p->longest_seq / 2) return false;
    return resident_of<bwd_kernel<D, PAIRS>>(128 * PAIRS) > 0;
}
bool is_one(const skrull_attn_plan_t *p)
{
    if (p->d == 128) return is_one<128, PAIRS_8W>(p);
    return dkv_pairs(p) == PAIRS_12W ? is_one<64, PAIRS_12W>(p) : is_one<64, PAIRS_8W>(p);
}

// The work items of dQ in one launch with dK/dV, where dK/dV begins on the compute units that dQ leaves.  Few long units, which a
// dQ launch of its own would wait for, are no longer what counts; the row blocks of a KV group are then
// better put together, as many as a workgroup has wavefronts, on fewer compute units, unless dQ leaves half of the chip
// anyway.  At head_dim 64 see skrull_attn_plan::dq_packed; at 128 this is for what runs at once (else they are put together in
// any case): of 50 backwards of 500 to 4,400 tokens 16 take 2 to 13 % less time, the others within 1 % of the same.  Units for workgroups of 4, more than there are larger ones at once, are made as large as these: 560 such units
// took two rounds (4,925 tokens in 10 sequences, 14/2 heads: backward 61 us, 58 as two launches, 43 with units of 12).
RowLaunch rows_dq_first(const skrull_attn_plan_t *p)
{
    const RowLaunch alone = rows_dq_alone(p);
    if (p->d == 128) {
        if (!p->units[1] || p->Hq == p->Hkv || 2 * alone.n_work <= resident_of<bwd_kernel<128, PAIRS_8W>>(128 * PAIRS_8W)) return alone;
        return row_launch<dq_kernel<128, NWQ_LARGE>>(p, NWQ_LARGE, true);
    }
    const bool wide = dkv_pairs(p) == PAIRS_12W;
    const int at_once = wide ? resident_of<bwd_kernel<64, PAIRS_12W>>(128 * PAIRS_12W) : resident_of<bwd_kernel<64, PAIRS_8W>>(128 * PAIRS_8W);
    if (wide && p->dq_packed && 2 * alone.n_work > at_once) return row_launch<dq_kernel<64, NWQ_WIDE>>(p, NWQ_WIDE, true);
    if (p->dq_waves == NWQ_SMALL && !p->dq_piped && alone.n_work > at_once)
        return wide ? row_launch<dq_kernel<64, NWQ_WIDE>>(p, NWQ_WIDE) : row_launch<dq_kernel<64, NWQ_LARGE>>(p, NWQ_LARGE);
    return alone;
}

template <int D, auto KernelQ, auto KernelKV>
hipError_t launch_pair(const skrull_attn_plan_t *p, BwdParams prm, int threads_q, int threads_kv, hipStream_t st,
                       hipEvent_t *ev)
{
    // dQ first: it also leaves -D and LSE*log2(e) of every (head, row) in the workspace,
    // which dK/dV reads.  Events: ev[0] start, ev[1] after dQ, ev[2] after dK/dV.
    if (ev) (void)hipEventRecord(ev[0], st);
    const bool queued_q = wants_queue<KernelQ>(threads_q, prm.n_work_dq), queued_kv = wants_queue<KernelKV>(threads_kv, prm.n_work_dkv);
    if ((queued_q || queued_kv) && !prm.clear) {
        queue_reset_kernel<<<1, 64, 0, st>>>(prm.queue_dq, 2, prm.queue_stride);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (!queued_q) prm.queue_dq = nullptr;
    if (!queued_kv) prm.queue_dkv = nullptr;
    KernelQ<<<launch_size<KernelQ>(threads_q, prm.n_work_dq, queued_q), threads_q, 0, st>>>(prm);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (ev) (void)hipEventRecord(ev[1], st);
    KernelKV<<<launch_size<KernelKV>(threads_kv, prm.n_work_dkv, queued_kv), threads_kv, 0, st>>>(prm);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p->n_split > 0) {
        const dim3 grid((unsigned)p->n_split * p->Hkv, (unsigned)(p->BN + REDUCE_ROWS<D> - 1) / REDUCE_ROWS<D>, 2);
        dkv_reduce_kernel<D><<<grid, 256, 0, st>>>(prm);
        e = hipGetLastError();
    }
    if (e == hipSuccess && ev) (void)hipEventRecord(ev[2], st);
    return e;
}

template <int D, int PAIRS>
hipError_t launch_one(const skrull_attn_plan_t *p, const BwdParams &prm, hipStream_t st)
{
    const int64_t work = (int64_t)prm.n_work_dq + prm.n_work_dkv;
    const int resident = resident_of<bwd_kernel<D, PAIRS>>(128 * PAIRS);
    bwd_kernel<D, PAIRS><<<(int)(work < resident ? work : resident), 128 * PAIRS, 0, st>>>(prm);
    return hipGetLastError();
}
template <int D>
hipError_t launch_d(const skrull_attn_plan_t *p, const BwdParams &prm, bool one, hipStream_t st, hipEvent_t *ev)
{
    if (one) {
        if constexpr (D == 64)
            if (dkv_pairs(p) == PAIRS_12W) return launch_one<D, PAIRS_12W>(p, prm, st);
        return launch_one<D, PAIRS_8W>(p, prm, st);
    }
    if constexpr (D == 64) {  // dQ has its other shapes, and dK/dV its 12-wavefront one, only here
        if (dkv_pairs(p) == PAIRS_12W) {
            if (p->dq_waves == NWQ_SMALL && p->dq_piped) return launch_pair<D, dq_kernel<D, NWQ_SMALL, true>, dkv_kernel<D, PAIRS_12W>>(p, prm, 64 * NWQ_SMALL, 128 * PAIRS_12W, st, ev);
            if (p->dq_waves == NWQ_SMALL) return launch_pair<D, dq_kernel<D, NWQ_SMALL>, dkv_kernel<D, PAIRS_12W>>(p, prm, 64 * NWQ_SMALL, 128 * PAIRS_12W, st, ev);
            if (p->dq_waves == NWQ_WIDE) return launch_pair<D, dq_kernel<D, NWQ_WIDE>, dkv_kernel<D, PAIRS_12W>>(p, prm, 64 * NWQ_WIDE, 128 * PAIRS_12W, st, ev);
            return launch_pair<D, dq_kernel<D, NWQ_LARGE>, dkv_kernel<D, PAIRS_12W>>(p, prm, 64 * NWQ_LARGE, 128 * PAIRS_12W, st, ev);
        }
        if (p->dq_waves == NWQ_SMALL && p->dq_piped) return launch_pair<D, dq_kernel<D, NWQ_SMALL, true>, dkv_kernel<D, PAIRS_8W>>(p, prm, 64 * NWQ_SMALL, 128 * PAIRS_8W, st, ev);
        if (p->dq_waves == NWQ_SMALL) return launch_pair<D, dq_kernel<D, NWQ_SMALL>, dkv_kernel<D, PAIRS_8W>>(p, prm, 64 * NWQ_SMALL, 128 * PAIRS_8W, st, ev);
        if (p->dq_waves == NWQ_WIDE) return launch_pair<D, dq_kernel<D, NWQ_WIDE>, dkv_kernel<D, PAIRS_8W>>(p, prm, 64 * NWQ_WIDE, 128 * PAIRS_8W, st, ev);
    }
    return launch_pair<D, dq_kernel<D, NWQ_LARGE>, dkv_kernel<D, PAIRS_8W>>(p, prm, 64 * NWQ_LARGE, 128 * PAIRS_8W, st, ev);
}

}  // namespace

int grid_dq(const skrull_attn_plan_t *p) { return rows_dq_alone(p).n_work; }

static KeyMap map_dkv(const skrull_attn_plan_t *p)
{
    const int SUB = 32 * dkv_pairs(p), passes = (p->BN + SUB - 1) / SUB;
    return KeyMap{p->BN, p->Hq / p->Hkv, passes, p->Hkv, p->n_split, p->n_whole_first, p->split_parts, p->split_chain,
                  p->split_compact ? p->n_split * p->BN : 0, inverse_of(passes), inverse_of(p->Hkv), p->dkv_units,
                  inverse_of(passes * p->Hkv)};
}

int grid_dkv(const skrull_attn_plan_t *p)
{
    const int n = p->dkv_units ? p->n_dkv_units : p->n_dkv + p->n_split * (p->split_parts - 1);
    return n * p->Hkv * map_dkv(p).passes;
}

hipError_t launch_bwd(const skrull_attn_plan_t *p, const void *q, const void *k, const void *v,
                      const void *o, const float *lse, const void *d_o, void *dq, void *dk,
                      void *dv, float *delta, hipStream_t st, hipEvent_t *ev, WgTrace *trace)
{
    BwdParams prm;
    prm.trace_dq = trace;
    DefaultStream &own = *p->default_stream;
    std::unique_lock<std::mutex> held(own.lock);
    bool in_turn = own.has(st);
    // Events are to time dQ and dK/dV by themselves.  Calls without a set of the plan's have the 256 bytes in the workspace alone for what
    // workgroups share, two lines, and workgroups that wait would poll the line of dQ's queues: replayed from a graph, 838 tokens in 10
    // sequences, 32/8 heads of 128, 39 us as three launches, 74 in one; 17,205 in 62, 8/4 heads, 204 and 295.
    const bool one = in_turn && !ev && is_one(p);
    const RowLaunch rows_q = one ? rows_dq_first(p) : rows_dq_alone(p);
    in_turn = in_turn && (one || rows_q.queued || dkv_queued(p));  // (two plain grids share nothing)
    if (!in_turn) held.unlock();
    prm.trace_dkv = trace ? trace + grid_dq(p) : nullptr;  // (one launch has as many dQ items or fewer)
    prm.q = (const uint16_t *)q; prm.k = (const uint16_t *)k; prm.v = (const uint16_t *)v;
    prm.d_o = (const uint16_t *)d_o; prm.o = (const uint16_t *)o; prm.lse = lse; prm.delta = delta;
    prm.lse2 = delta + (size_t)p->Hq * p->total_q;
    prm.dq = (uint16_t *)dq; prm.dk = (uint16_t *)dk; prm.dv = (uint16_t *)dv;
    prm.fwd_items = (const int4 *)p->fwd_items; prm.dkv_items = (const int4 *)p->dkv_items;
    prm.cu_q = p->cu_q; prm.cu_k = p->cu_k; prm.q_begin = p->q_begin; prm.q_len = p->q_len;
    prm.kv_len = p->kv_len; prm.shares_kv = p->shares_kv;
    prm.Hq = p->Hq; prm.Hkv = p->Hkv; prm.total_q = p->total_q;
    prm.rows = rows_q.rows;
    prm.keys = map_dkv(p);
    prm.scale = p->scale; prm.scale_log2 = p->scale * kLog2e;
    prm.total_k = p->total_k;
    prm.n_work_dq = rows_q.n_work;
    prm.n_work_dkv = grid_dkv(p);
    {
        // workspace: -D | LSE*log2e | (256-byte aligned) 256 bytes, the queues of calls that clear them first | dK partials | dV partials
        static_assert(2 * 8 * kQueueStrideWorkspace * sizeof(WorkQueue) == 256, "the queues' part of the workspace");
        static_assert(2 * 8 * kQueueStride * sizeof(WorkQueue) == 2 * 4 * SKRULL_QUEUE_INTS, "the queues' part of a plan's state");
        const size_t rows = (((size_t)p->Hq * p->total_q * 8) + 255) & ~(size_t)255;
        prm.dk_part = (float *)((char *)delta + rows + 256);
        const size_t part_rows = p->split_compact ? (size_t)p->n_split * p->BN : (size_t)p->total_k;
        prm.dv_part = prm.dk_part + (size_t)p->split_parts * part_rows * p->Hkv * p->d;
    }
    prm.n_parts = 0;
    if ((int64_t)p->n_split * p->Hkv > SKRULL_ITEM_COUNTERS)
        prm.n_parts = (p->dkv_units ? p->n_dkv_units - (p->n_dkv - p->n_split) : p->n_split * p->split_parts) * p->Hkv * prm.keys.passes;
    if (in_turn) {
        int32_t *sets = p->sets + 2 * SKRULL_QUEUE_INTS, *mine = sets + (own.bwd & 1) * SKRULL_BWD_STATE_INTS;
        prm.queue_stride = kQueueStride;
        prm.queue_dq = (WorkQueue *)mine;
        prm.queue_dkv = (WorkQueue *)(mine + SKRULL_QUEUE_INTS);
        prm.rows_ready = mine + 2 * SKRULL_QUEUE_INTS;
        prm.next_sum = prm.rows_ready + 32;
        prm.parts_stored = prm.rows_ready + (prm.n_parts ? 64 : 128);
        prm.clear = sets + (~own.bwd & 1) * SKRULL_BWD_STATE_INTS;
    } else {
        prm.queue_stride = kQueueStrideWorkspace;
        prm.queue_dq = (WorkQueue *)((char *)prm.dk_part - 256);
        prm.queue_dkv = prm.queue_dq + 8 * kQueueStrideWorkspace;
        prm.rows_ready = prm.parts_stored = prm.next_sum = prm.clear = nullptr;
    }
    const hipError_t e = p->d == 128 ? launch_d<128>(p, prm, one, st, ev) : p->d == 64 ? launch_d<64>(p, prm, one, st, ev) : hipErrorInvalidValue;
    if (in_turn) {
        if (e == hipSuccess) ++own.bwd;
        else own.lost = true;
    }
    return e;
}
