"""autograd.skrull_attention in native code against the Function of the same module, which takes the calls that something
watches from Python: same bits, same errors, same treatment of the plan and of what is saved for the backward."""
import gc

import pytest
import torch

pytestmark = pytest.mark.gpu


def _case(S=(70, 1, 300), heads=(4, 2), d=64):
    from paper_2505_19609_amd import binding as B
    plan = B.skrull_attn_plan(list(S), [1] * len(S), [0] * len(S), heads[0], heads[1], d, d ** -0.5)
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v, do = (torch.randn(shape, generator=gen, device="cuda").bfloat16() for shape in
                   ((sum(S), heads[0], d), (sum(S), heads[1], d), (sum(S), heads[1], d), (sum(S), heads[0], d)))
    return plan, [t.requires_grad_() for t in (q, k, v)], do


def _both(monkeypatch, f):
    from paper_2505_19609_amd import autograd as A
    out = []
    for watched in (True, False):
        monkeypatch.setattr(A, "_watched", lambda: watched)
        out.append(f(A.skrull_attention))
    assert A._native   # (else both were the Function)
    return out


@pytest.mark.parametrize("heads,d", [((4, 2), 64), ((28, 4), 128)])
def test_same_bits(monkeypatch, heads, d):
    plan, qkv, do = _case(heads=heads, d=d)

    def run(attention):
        o = attention(*qkv, plan)
        grads = torch.autograd.grad(o, qkv, do, retain_graph=True)
        again = torch.autograd.grad(o, qkv, do.transpose(0, 1).contiguous().transpose(0, 1))   # (another layout of dO)
        with torch.no_grad():
            assert not attention(*qkv, plan).requires_grad
        return (o.detach(), *grads, *again)

    for a, b in zip(*_both(monkeypatch, run)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    plan.destroy()


def test_saved_tensors_go_through_hooks(monkeypatch):
    plan, qkv, do = _case()

    def run(attention):
        packed = []
        with torch.autograd.graph.saved_tensors_hooks(lambda t: packed.append(t.shape) or t.cpu(), lambda t: t.cuda()):
            o = attention(*qkv, plan)
        return packed, torch.autograd.grad(o, qkv, do)

    (p0, g0), (p1, g1) = _both(monkeypatch, run)
    assert p0 == p1 and len(p0) == 5
    assert all(torch.equal(a, b) for a, b in zip(g0, g1))
    plan.destroy()


def test_errors(monkeypatch):
    from paper_2505_19609_amd import binding as B
    plan, qkv, do = _case()
    q, k, v = qkv

    def run(attention):
        for args in ((q[1:], k, v), (q, k[:, :1].contiguous(), v), (q, k, v[:-1]), (q.float(), k, v), (q, k.transpose(0, 1), v)):
            with pytest.raises(ValueError):
                attention(*args, plan)
        o = attention(*qkv, plan)
        o.backward(do)
        with pytest.raises(RuntimeError, match="second time"):
            o.backward(do)
        o = attention(*qkv, plan)
        with torch.no_grad():
            q.add_(1)                          # what the backward needs has changed
        with pytest.raises(RuntimeError, match="inplace"):
            o.backward(do)
        dead = B.skrull_attn_plan([371], [1], [0], 4, 2, 64, 0.125)
        o = attention(*qkv, dead)
        dead.destroy()
        with pytest.raises(B.SkrullError) as e:   # destroyed between forward and backward
            o.backward(do)
        assert e.value.code == B.SKRULL_EINVAL
        with pytest.raises(B.SkrullError):
            attention(*qkv, dead)
        return True

    assert _both(monkeypatch, run) == [True, True]
    plan.destroy()


def test_the_graph_keeps_the_plan(monkeypatch):
    from paper_2505_19609_amd.autograd import skrull_attention
    plan, qkv, do = _case()
    want = torch.autograd.grad(skrull_attention(*qkv, plan), qkv, do)

    def run(attention):
        mine, _, _ = _case()
        o = attention(*qkv, mine)
        del mine
        gc.collect()
        return torch.autograd.grad(o, qkv, do)

    for grads in _both(monkeypatch, run):
        assert all(torch.equal(a, b) for a, b in zip(grads, want))
    plan.destroy()


def test_traced_and_transformed_calls_take_the_function():
    from paper_2505_19609_amd.autograd import skrull_attention
    plan, qkv, do = _case()
    want = skrull_attention(*qkv, plan)
    traced = torch.jit.trace(lambda q, k, v: skrull_attention(q, k, v, plan) * 1, [t.detach() for t in qkv], check_trace=False)
    other = [t.detach().clone().mul_(0.5) for t in qkv]
    assert torch.equal(traced(*other), skrull_attention(*other, plan))   # (not the tensors it was traced with)
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda q: skrull_attention(q, *qkv[1:], plan).float().sum())(qkv[0])
    assert want.requires_grad
    plan.destroy()


@pytest.mark.parametrize("backend", ["eager", "aot_eager"])
def test_compiled_calls(backend):
    from paper_2505_19609_amd.autograd import skrull_attention
    plan, qkv, do = _case()
    want = torch.autograd.grad(skrull_attention(*qkv, plan) * 2, qkv, do)
    torch._dynamo.reset()
    got = torch.autograd.grad(torch.compile(lambda q, k, v: skrull_attention(q, k, v, plan) * 2, backend=backend)(*qkv), qkv, do)
    for a, b in zip(got, want):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    plan.destroy()
