// Host side of skrull_attn_plan against a runtime made of the functions below: what becomes of the pinned memory through
// which a plan's kernels talk to the host, when calls of the runtime fail.  Compiled for the host only; no GPU, no HIP library.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <set>
#include <string>

#include "common.h"

namespace {
std::set<const void *> in_flight;  // slots that a kernel which may still run reads and writes
const void *last_slot = nullptr;   // slot of the last launch that had one
const char *pinned = nullptr;
size_t pinned_bytes = 0;
int fail_units = 0, host_allocations_to_fail = 0;
unsigned int host_flags = 0;         // of the last allocation of pinned memory
bool waits_fail = false;
bool other_thread_plans = false;   // a plan is made by another thread while this one frees memory

[[noreturn]] void fail(const char *what)
{
    printf("%s\n", what);
    exit(1);
}
void expect(bool ok, const char *what) { if (!ok) fail(what); }

void launched(const void *slot)
{
    const char *at = (const char *)slot;
    if (at < pinned || at >= pinned + pinned_bytes) return;
    last_slot = slot;
    if (!in_flight.insert(slot).second) fail("a slot was handed out that a kernel still uses");
}
hipError_t wait()
{
    if (waits_fail) return hipErrorUnknown;
    in_flight.clear();
    return hipSuccess;
}
int plan(int tokens)
{
    const int32_t S = tokens, one = 1, zero = 0;
    skrull_attn_problem_t p = {};
    p.num_seqs = 1; p.seq_len = &S; p.shard_degree = &one; p.shard_index = &zero;
    p.num_q_heads = 4; p.num_kv_heads = 2; p.head_dim = 64; p.softmax_scale = 0.125f; p.block_m = p.block_n = 64;
    skrull_attn_plan_t *out = nullptr;
    const int rc = skrull_attn_plan(&p, nullptr, &out);
    skrull_attn_plan_destroy(out);
    return rc;
}
constexpr int kOneWorkgroup = 1000, kSeveralKernels = 64 * 600;  // tokens
void totals_of(PlanTotals *t, int rows)
{
    memset(t, 0, sizeof *t);
    t->total_q = t->total_k = rows;
    t->n_fwd = t->n_dkv = (rows + 63) / 64;
    t->n_seg = 1;
    t->block_n = 64;
    t->split.parts = t->split.head_split = 1;
}
}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "made to fail"; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) { static char s; *p = &s; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = malloc(n); return hipSuccess; }
hipError_t hipFree(void *p)
{
    if (other_thread_plans) {
        other_thread_plans = false;
        expect(plan(kOneWorkgroup) == SKRULL_OK, "the other thread's plan failed");
    }
    (void)wait();  // (for the whole device)
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned int flags)
{
    host_flags = flags;
    if (host_allocations_to_fail > 0) { --host_allocations_to_fail; return hipErrorStreamCaptureUnsupported; }
    *p = malloc(n);
    pinned = (const char *)*p;
    pinned_bytes = n;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return wait(); }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
}

hipError_t launch_plan_small(const SmallPlan &j, hipStream_t)
{
    launched(j.in);
    totals_of(j.totals, j.in[0]);
    return hipSuccess;
}
hipError_t launch_plan_ranges(const int32_t *S, const int32_t *, const int32_t *, const int32_t *, int32_t, int32_t, int32_t, int32_t,
                              int32_t, int32_t *, int32_t *, int32_t *, int32_t *, int32_t *, int32_t *, int32_t *, int32_t *,
                              int32_t, int32_t, int32_t, int32_t, int32_t, PlanTotals *totals, hipStream_t)
{
    launched(S);
    totals_of(totals, S[0]);
    return hipSuccess;
}
hipError_t launch_plan_items(const skrull_attn_plan_t *, const int32_t *, const int32_t *, int32_t, int32_t, int32_t *, int32_t *,
                             int32_t *, int32_t, int32_t, PlanTotals *, hipStream_t) { return hipSuccess; }
hipError_t launch_plan_units(const skrull_attn_plan_t *, int32_t, int32_t, int32_t, int32_t, int32_t, PlanTotals *, hipStream_t)
{
    if (fail_units > 0) { --fail_units; return hipErrorUnknown; }
    return hipSuccess;
}
int64_t plan_dkv_unit_ints(const skrull_attn_plan_t *, int32_t, int32_t) { return 0; }
int64_t plan_unit_ints(const skrull_attn_plan_t *, int32_t, int) { return 0; }
int64_t plan_radix_ints(int32_t, int32_t, int32_t) { return 0; }

int main(int, char **argv)
{
    const std::string what = argv[1];
    if (what == "wait_fails") {  // nobody knows when the kernel is done
        waits_fail = true;
        expect(plan(kOneWorkgroup) != SKRULL_OK, "the call hid a failed wait");
        waits_fail = false;
        std::set<const void *> kept = in_flight;
        for (int i = 0; i < 40; ++i) {
            in_flight = kept;
            expect(plan(kOneWorkgroup) == SKRULL_OK && last_slot, "a later plan failed");
        }
    } else if (what == "launch_fails") {  // kernels of the call are queued already
        fail_units = 1;
        other_thread_plans = true;
        expect(plan(kSeveralKernels) != SKRULL_OK, "the call hid a failed launch");
        expect(!other_thread_plans, "no other plan was made");
    } else if (what == "failures_use_up_no_slots") {
        for (fail_units = 40; fail_units > 0;) expect(plan(kSeveralKernels) != SKRULL_OK, "the call hid a failed launch");
        expect(plan(kOneWorkgroup) == SKRULL_OK && last_slot, "a plan failed after failures of others");
        for (int i = 0; i < 40; ++i) {
            last_slot = nullptr;
            expect(plan(i % 2 ? kOneWorkgroup : kSeveralKernels) == SKRULL_OK && last_slot, "no slot left");
        }
    } else if (what == "memory_is_coherent") {  // whatever the environment says about memory that does not ask
        expect(plan(kOneWorkgroup) == SKRULL_OK && last_slot, "a plan failed");
        expect(host_flags & hipHostMallocCoherent, "kernels and the host share memory that is not coherent");
        expect(host_flags & hipHostMallocPortable, "the memory is one device's only");
    } else if (what == "memory_comes_later") {  // for instance another thread was capturing a graph
        host_allocations_to_fail = 3;
        for (int i = 0; i < 3; ++i) {
            expect(plan(kSeveralKernels) == SKRULL_OK && !last_slot, "a plan failed without pinned memory");
        }
        expect(host_allocations_to_fail == 0, "the memory was not asked for again");
        expect(plan(kOneWorkgroup) == SKRULL_OK && last_slot, "no slot after the memory came");
    } else {
        fail("unknown case");
    }
    return 0;
}
