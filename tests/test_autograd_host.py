"""autograd.skrull_attention without a GPU: what it refuses is refused with the same error by its native code and by the
Function that takes the calls which something watches from Python."""
import pytest
import torch

from paper_2505_19609_amd import autograd as A
from paper_2505_19609_amd import binding as B


def _plan(tq=3, tk=3, hq=2, hkv=1, d=64):
    return B.Plan(None, B.PlanInfo(total_q=tq, total_k=tk, num_q_heads=hq, num_kv_heads=hkv, head_dim=d))


@pytest.mark.parametrize("watched", [False, True])
def test_refused_the_same_way_by_both_paths(monkeypatch, watched):
    monkeypatch.setattr(A, "_watched", lambda: watched)
    q, k = torch.zeros(3, 2, 64, dtype=torch.bfloat16), torch.zeros(3, 1, 64, dtype=torch.bfloat16)
    for args in ((q, k, k), (q.float(), k, k), (q, k.transpose(0, 1), k)):   # on the CPU, of another type, not contiguous
        with pytest.raises(ValueError, match="contiguous bf16 CUDA tensors"):
            A.skrull_attention(*args, _plan())
    with pytest.raises(AttributeError):
        A.skrull_attention(None, k, k, _plan())
    assert (A._native is not None) or watched


def test_watched_calls_are_seen():
    assert not A._watched()
    with torch.autograd.forward_ad.dual_level():
        assert A._watched()
    seen = []

    def f(x):
        seen.append(A._watched())
        return x * 2

    torch.func.vmap(f)(torch.zeros(2))
    torch.jit.trace(f, torch.zeros(2), check_trace=False)
    assert seen == [True, True]
