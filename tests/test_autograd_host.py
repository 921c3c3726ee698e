"""autograd.skrull_attention without a GPU: what it refuses is refused with the same error by its native code and by the
Function that takes the calls which something watches from Python."""
import sys
import warnings

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


@pytest.mark.parametrize("why", ["missing", "another_torch"])
def test_without_the_native_module_calls_take_the_function(monkeypatch, why):
    import paper_2505_19609_amd as package
    monkeypatch.setattr(A, "_native", None)
    monkeypatch.delattr(package, "_autograd", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2505_19609_amd._autograd", None)   # (an import raises ImportError)
    if why == "another_torch":
        class Broken:
            def find_spec(self, name, path=None, target=None):
                if name == "paper_2505_19609_amd._autograd":
                    raise ImportError("undefined symbol")
        monkeypatch.delitem(sys.modules, "paper_2505_19609_amd._autograd")
        monkeypatch.setattr(sys, "meta_path", [Broken(), *sys.meta_path])
    taken = []
    monkeypatch.setattr(A._SkrullAttention, "apply", lambda *args: taken.append(args) or "o")
    q, k, plan = torch.zeros(3, 2, 64, dtype=torch.bfloat16), torch.zeros(3, 1, 64, dtype=torch.bfloat16), _plan()
    with pytest.warns(RuntimeWarning, match="cannot be loaded"):
        assert A.skrull_attention(q, k, k, plan) == "o"
    with warnings.catch_warnings():
        warnings.simplefilter("error")      # (said once)
        assert A.skrull_attention(q, k, k, plan) == "o"
    assert len(taken) == 2 and taken[0][3] is plan


def test_the_library_is_built_without_torch(monkeypatch):
    from paper_2505_19609_amd import build
    ran = []
    monkeypatch.setattr(build, "find_spec", lambda name: None)
    monkeypatch.setattr(build, "_compile", lambda src: src + ".o")
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **kw: ran.append(cmd))
    assert build.build_library() == build.LIB
    assert len(ran) == 1 and ran[0][0] == "hipcc" and build.LIB in ran[0]
