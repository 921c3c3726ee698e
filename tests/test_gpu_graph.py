"""The forward and backward entry points only enqueue kernels on the caller's stream
(no allocation, no memset, no synchronisation), so a launch-bound inner loop can be
captured in a HIP graph.  Capture one forward + backward, replay it several times with
eager work and synchronisations in between, and compare every replay bit for bit with
the eager result on the same inputs."""
import numpy as np
import pytest
import torch

from paper_2505_19609_amd import workloads as W
from gpu_util import to_dev, dkv_begins_during_dq

pytestmark = pytest.mark.gpu


SMALL = ([700, 129, 2100, 64], [1, 1, 3, 1], [0, 0, 1, 0], [0, 0, 1, 0])
# more work items than the chip holds workgroups at once: the persistent launches with their
# work queues (and the kernels that clear them) are what is captured
LARGE = ([9000, 700, 6100, 64], [1, 1, 3, 1], [0, 0, 1, 0], [0, 0, 1, 0])


@pytest.mark.parametrize("heads,d,split,lengths", [((4, 2), 64, 0, SMALL), ((14, 2), 64, 3, SMALL), ((8, 2), 128, 1, SMALL),
                                                   ((16, 4), 128, 1, LARGE), ((14, 2), 64, 0, LARGE)])
def test_graph_replays_equal_eager(heads, d, split, lengths):
    from paper_2505_19609_amd import binding as B
    w = W.Workload("graph", lengths[0], lengths[1], lengths[2], heads[0], heads[1], d,
                   d ** -0.5, 4321, shard_cut=lengths[3])
    plan = B.skrull_attn_plan(w.seq_len, w.shard_degree, w.shard_index, heads[0], heads[1], d,
                              w.softmax_scale, shard_cut=w.shard_cut, head_split=split)
    vals = W.make_values(w, plan.total_q, plan.total_k)
    dev = {n: to_dev(a) for n, a in vals.items()}
    outs = {n: torch.empty_like(dev[src]) for n, src in (("o", "q"), ("dq", "q"), ("dk", "k"), ("dv", "k"))}
    lse = torch.empty((heads[0], plan.total_q), dtype=torch.float32, device="cuda")
    ws = torch.empty(max(int(plan.bwd_workspace_bytes), 16), dtype=torch.uint8, device="cuda")

    def step():
        B.skrull_attn_fwd(plan, dev["q"], dev["k"], dev["v"], outs["o"], lse)
        B.skrull_attn_bwd(plan, dev["q"], dev["k"], dev["v"], outs["o"], lse, dev["do"],
                          outs["dq"], outs["dk"], outs["dv"], ws)

    step()
    torch.cuda.synchronize()
    eager = {n: t.clone() for n, t in outs.items()}
    eager["lse"] = lse.clone()

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):   # warm-up on the capture stream
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for rep in range(4):
        for t in list(outs.values()) + [lse, ws]:
            t.view(torch.uint8).fill_(0xFF if rep % 2 else 0)   # the program's own eager work in between
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for n, t in outs.items():
            assert torch.equal(t, eager[n]), (rep, n)
        assert torch.equal(lse, eager["lse"]), rep
    plan.destroy()


def test_forward_calls_of_one_plan_overlap_on_two_streams():
    """A plan's forward calls take the plan's work-queue slots in turn, so calls that overlap on
    different streams do not share a queue: two streams run the same plan's forward at the same
    time, several times over, and every output equals the one-stream result bit for bit."""
    from paper_2505_19609_amd import binding as B
    heads, d = (16, 4), 128
    w = W.Workload("two_streams", [9000, 700, 4000], [1, 1, 1], [0, 0, 0], heads[0], heads[1], d, d ** -0.5, 99)
    plan = B.skrull_attn_plan(w.seq_len, w.shard_degree, w.shard_index, heads[0], heads[1], d, w.softmax_scale)
    first, num = B.skrull_attn_trace_layout(plan)
    assert num[0] > 256          # more work items than compute units: the launch is persistent
    vals = W.make_values(w, plan.total_q, plan.total_k)
    dev = {n: to_dev(a) for n, a in vals.items()}
    ref_o = torch.empty_like(dev["q"])
    ref_lse = torch.empty((heads[0], plan.total_q), dtype=torch.float32, device="cuda")
    B.skrull_attn_fwd(plan, dev["q"], dev["k"], dev["v"], ref_o, ref_lse)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [(torch.empty_like(ref_o), torch.empty_like(ref_lse)) for _ in streams]
    for rep in range(40):        # wraps around the plan's 64 slots
        for st, (o, lse) in zip(streams, outs):
            if rep % 8 == 0:
                o.fill_(float("nan")); lse.fill_(float("nan"))
            st.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(st):
                B.skrull_attn_fwd(plan, dev["q"], dev["k"], dev["v"], o, lse)
        if rep % 8 == 7:
            torch.cuda.synchronize()
            for o, lse in outs:
                assert torch.equal(o.view(torch.int16), ref_o.view(torch.int16)), rep
                assert torch.equal(lse, ref_lse), rep
    torch.cuda.synchronize()
    plan.destroy()


@pytest.mark.parametrize("heads,d,S", [((16, 4), 128, [9000, 700, 4000]), ((14, 2), 64, [700] * 30 + [64])])
def test_calls_of_one_plan_on_many_streams_and_in_graphs_by_turns(heads, d, S):
    """A launch on the default stream clears the queues that the next one uses; calls on other streams and captured ones
    clear a queue first.  All by turns, on one plan, overlapping: every result is the same bits."""
    from paper_2505_19609_amd import binding as B
    w = W.Workload("many_streams", S, [1] * len(S), [0] * len(S), heads[0], heads[1], d, d ** -0.5, 98)
    plan = B.skrull_attn_plan(S, [1] * len(S), [0] * len(S), heads[0], heads[1], d, w.softmax_scale)
    assert all(n > 256 for n in B.skrull_attn_trace_layout(plan)[1])  # persistent launches
    dev = {n: to_dev(a) for n, a in W.make_values(w, plan.total_q, plan.total_k).items()}

    def outputs():
        return {"o": torch.empty_like(dev["q"]), "lse": torch.empty((heads[0], plan.total_q), dtype=torch.float32, device="cuda"),
                "dq": torch.empty_like(dev["q"]), "dk": torch.empty_like(dev["k"]), "dv": torch.empty_like(dev["v"]),
                "ws": torch.empty(int(plan.bwd_workspace_bytes), dtype=torch.uint8, device="cuda")}

    def step(t):
        B.skrull_attn_fwd(plan, dev["q"], dev["k"], dev["v"], t["o"], t["lse"])
        B.skrull_attn_bwd(plan, dev["q"], dev["k"], dev["v"], t["o"], t["lse"], dev["do"], t["dq"], t["dk"], t["dv"], t["ws"])

    ref = outputs()
    step(ref)
    streams = [torch.cuda.default_stream()] + [torch.cuda.Stream() for _ in range(5)]   # (60 forward calls with a slot, below: a plan has 64)
    outs = [outputs() for _ in streams]
    captured, graph = outputs(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=streams[1]):
        step(captured)
    for rep in range(6):
        for t in outs + [captured]:
            for x in t.values():
                x.view(torch.uint8).fill_(0xFF if rep % 2 else 0)
        torch.cuda.synchronize()
        for k in range(2):
            for i, (st, t) in enumerate(zip(streams, outs)):
                with torch.cuda.stream(st):
                    step(t)
                    if k == 0 and i == rep:
                        graph.replay()
        torch.cuda.synchronize()
        for t in outs + [captured]:
            for n in ("o", "lse", "dq", "dk", "dv"):
                assert torch.equal(t[n].view(torch.uint8), ref[n].view(torch.uint8)), (rep, n)
    plan.destroy()


@pytest.mark.parametrize("where", ["default", "graph", "stream"])
def test_only_calls_on_the_default_stream_are_one_launch(where):
    """dK/dV begins while dQ is under way on the default stream, whose calls have queues in the plan.  A captured backward
    makes them launches of their own (in one, with the workspace's queues, it took up to twice as long), and so does one on a
    stream that the program made: its handle may stand for another stream later, with the first one's work still
    under way, so the plan keeps nothing for it.  Same bits."""
    from paper_2505_19609_amd import binding as B
    S, heads, d = [277] * 62, (8, 4), 128
    w = W.Workload("launches", S, [1] * len(S), [0] * len(S), heads[0], heads[1], d, d ** -0.5, 97)
    plan = B.skrull_attn_plan(S, [1] * len(S), [0] * len(S), heads[0], heads[1], d, w.softmax_scale)
    dev = {n: to_dev(a) for n, a in W.make_values(w, plan.total_q, plan.total_k).items()}
    o, lse = torch.empty_like(dev["q"]), torch.empty((heads[0], plan.total_q), device="cuda")
    outs = [[torch.empty_like(dev[n]) for n in "qkv"] for _ in range(2)]
    ws = torch.empty(max(int(plan.bwd_workspace_bytes), 16), dtype=torch.uint8, device="cuda")

    def backward(out):
        B.skrull_attn_bwd(plan, dev["q"], dev["k"], dev["v"], o, lse, dev["do"], *out, ws)

    B.skrull_attn_fwd(plan, dev["q"], dev["k"], dev["v"], o, lse)
    backward(outs[0])
    stream = torch.cuda.Stream()

    def call():
        if where == "graph":
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                backward(outs[1])
            graph.replay()
        elif where == "stream":
            with torch.cuda.stream(stream):
                backward(outs[1])
        else:
            backward(outs[1])

    assert dkv_begins_during_dq(plan, call) == (where == "default")
    for a, b in zip(*outs):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    plan.destroy()
