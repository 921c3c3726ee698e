"""The opt-in per-workgroup trace (a measurement aid): every workgroup that has work writes one
record, results do not change, and a buffer that is too small is refused."""
import numpy as np
import pytest

from paper_2505_19609_amd import workloads as W
from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
def test_trace_records_every_workgroup_and_changes_nothing(d):
    import torch
    from paper_2505_19609_amd import binding as B
    from paper_2505_19609_amd.balance import REC, analyse
    w = W.Workload("trace", [3000, 129, 700, 2100], [1, 1, 1, 3], [0, 0, 0, 1], 8, 2, d, d ** -0.5, 17)
    plan = B.skrull_attn_plan(w.seq_len, w.shard_degree, w.shard_index, 8, 2, d, w.softmax_scale)
    vals = W.make_values(w, plan.total_q, plan.total_k)
    dev = {n: to_dev(a) for n, a in vals.items()}
    first, num = B.skrull_attn_trace_layout(plan)
    assert first == [0, num[0], num[0] + num[1]] and all(n > 0 for n in num)
    outs = []
    for traced in (False, True):
        o, dq = torch.empty_like(dev["q"]), torch.empty_like(dev["q"])
        dk, dv = torch.empty_like(dev["k"]), torch.empty_like(dev["k"])
        lse = torch.empty((8, plan.total_q), dtype=torch.float32, device="cuda")
        ws = torch.empty(max(int(plan.bwd_workspace_bytes), 16), dtype=torch.uint8, device="cuda")
        records = torch.zeros((sum(num), REC.itemsize), dtype=torch.uint8, device="cuda")
        if traced:
            with pytest.raises(B.SkrullError):          # room for the forward only: the backward is refused
                B.skrull_attn_trace(records[:num[0]])
                B.skrull_attn_bwd(plan, dev["q"], dev["k"], dev["v"], o, lse, dev["do"], dq, dk, dv, ws)
            B.skrull_attn_trace(records)
        B.skrull_attn_fwd(plan, dev["q"], dev["k"], dev["v"], o, lse)
        B.skrull_attn_bwd(plan, dev["q"], dev["k"], dev["v"], o, lse, dev["do"], dq, dk, dv, ws)
        torch.cuda.synchronize()
        B.skrull_attn_trace(None)
        outs.append((o, lse, dq, dk, dv))
        if traced:
            rec = records.cpu().numpy().view(REC).reshape(-1)
            for f, n in zip(first, num):
                r = rec[f:f + n]
                r = r[r["one"] == 1]
                assert 0 < len(r) <= n
                assert (r["t1"] >= r["t0"]).all() and (r["t0"] > 0).all()
                assert len(np.unique(r["block"])) == len(r) and r["block"].max() < n
                a = analyse(r, 1)
                assert 0 < a["compute_units"] <= 256 and 0 < a["busy"] <= 1.0
        else:
            assert not records.any()
    for x, y in zip(*outs):
        assert torch.equal(x.view(torch.int16) if x.dtype == torch.bfloat16 else x,
                           y.view(torch.int16) if y.dtype == torch.bfloat16 else y)
    plan.destroy()


def test_profiling_switch_belongs_to_the_calling_thread():
    """One thread profiles, another does not: the second reads nothing back (SKRULL_EINVAL)
    and its calls record no events."""
    import threading
    import torch
    from paper_2505_19609_amd import binding as B
    w = W.config(1)
    plan = B.skrull_attn_plan(w.seq_len, w.shard_degree, w.shard_index, 4, 4, 64, 1.0)
    vals = W.make_values(w, plan.total_q, plan.total_k)
    dev = {n: to_dev(a) for n, a in vals.items()}
    o = torch.empty_like(dev["q"])
    lse = torch.empty((4, plan.total_q), dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    B.skrull_attn_profile(True)
    B.skrull_attn_fwd(plan, dev["q"], dev["k"], dev["v"], o, lse, stream=stream)
    seen = {}

    def other():
        torch.cuda.set_device(0)
        try:
            B.skrull_attn_profile_read()
        except B.SkrullError as e:
            seen["code"] = e.code
        B.skrull_attn_fwd(plan, dev["q"], dev["k"], dev["v"], o, lse, stream=stream)

    t = threading.Thread(target=other)
    t.start(); t.join()
    ms = B.skrull_attn_profile_read()
    B.skrull_attn_profile(False)
    torch.cuda.synchronize()
    assert seen.get("code") == B.SKRULL_EINVAL
    assert ms[0] > 0 and ms[2] == -1 and ms[3] == -1
    with pytest.raises(B.SkrullError):
        B.skrull_attn_profile_read()          # switched off again
    plan.destroy()


@pytest.mark.parametrize("what,d,wg", [("fwd", 128, 256), ("fwd", 64, 128), ("dq", 128, 256)])
def test_longest_items_start_first_beside_another_launch(what, d, wg):
    """Half of the compute units are held by another stream's launch when a forward / dQ with a work queue
    starts, so half of its workgroups start late.  The longest items, one for every workgroup of the launch,
    must not wait for those: on each die's list they begin before any item of its second half does."""
    import time
    import torch
    from paper_2505_19609_amd import binding as B
    from paper_2505_19609_amd.balance import REC

    def tensors(plan, hq, hkv, d):
        q, do = (torch.randn(plan.total_q, hq, d, device="cuda").bfloat16() for _ in range(2))
        k, v = (torch.randn(plan.total_k, hkv, d, device="cuda").bfloat16() for _ in range(2))
        return q, k, v, do, torch.empty_like(q), torch.empty((hq, plan.total_q), device="cuda")

    # 128 workgroups that fill a compute unit's LDS and run for over a millisecond
    hold = B.skrull_attn_plan([65536], [8], [7], 4, 1, 128, 128 ** -0.5, wg_query_rows=256)
    assert B.skrull_attn_trace_layout(hold)[1][0] == 128
    hq, hk, hv, _, ho, hlse = tensors(hold, 4, 1, 128)
    S = [1500] * 24 + [40] * 600
    plan = B.skrull_attn_plan(S, [1] * len(S), [0] * len(S), 8, 8, d, d ** -0.5, head_split=1, wg_query_rows=wg)
    q, k, v, do, o, lse = tensors(plan, 8, 8, d)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    ws = torch.empty(int(plan.bwd_workspace_bytes), dtype=torch.uint8, device="cuda")
    first, num = B.skrull_attn_trace_layout(plan)
    at = 0 if what == "fwd" else 1
    longest = 256 * (3 if wg == 128 else 1)         # workgroups that the empty chip holds at once
    for _ in range(4):                              # (two streams may share a hardware queue: then take others)
        records = torch.zeros((sum(num), REC.itemsize), dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        other, mine = torch.cuda.Stream(), torch.cuda.Stream()
        B.skrull_attn_fwd(plan, q, k, v, o, lse, stream=mine)  # (what a backward needs; a stream's first launch sets up its queue)
        B.skrull_attn_fwd(hold, hq, hk, hv, ho, hlse, stream=other)
        torch.cuda.synchronize()
        B.skrull_attn_fwd(hold, hq, hk, hv, ho, hlse, stream=other)
        time.sleep(2e-4)                            # (the other launch is under way)
        B.skrull_attn_trace(records)
        if what == "fwd":
            B.skrull_attn_fwd(plan, q, k, v, o, lse, stream=mine)
        else:
            B.skrull_attn_bwd(plan, q, k, v, o, lse, do, dq, dk, dv, ws, stream=mine)
        torch.cuda.synchronize()
        B.skrull_attn_trace(None)
        rec = records.cpu().numpy().view(REC).reshape(-1)[first[at]:first[at] + num[at]]
        assert (rec["one"] == 1).all()
        t0 = rec["t0"].astype(np.int64)
        t0 -= t0.min()
        unit = rec["xcc_id"].astype(np.int64) << 32 | rec["hw_id"] & 0xff00
        units = len(np.unique(unit[t0 < 2000]))
        print(f"{what} d {d}: {num[at]} items, on {units} compute units in the first 20 us; the longest {longest} begin by "
              f"{t0[:longest].max() / 100:.0f} us, the second half from {t0[num[at] // 2:].min() / 100:.0f} us on")
        if units <= 160:
            break
    else:
        pytest.skip("the two launches did not run side by side")
    for die in range(8):                            # (items die, die + 8, ... are one die's list)
        mine = t0[die::8]
        assert mine[:longest // 8].max() < mine[len(mine) // 2:].min(), die
    hold.destroy()
    plan.destroy()
