"""torch.autograd wrapper around the library's forward / backward, for callers that
train with PyTorch: argument marshalling and bookkeeping only, every step of the
attention runs in the HIP kernels behind the C ABI.  The marshalling is native code where
nothing watches the call from Python, else the Function below: the same checks, outputs and errors."""
from __future__ import annotations

import warnings

import torch

from . import binding as B


class _SkrullAttention(torch.autograd.Function):
    @staticmethod
    def forward(ctx, q, k, v, plan):
        if not (q.is_cuda and q.dtype == torch.bfloat16 and q.is_contiguous() and k.is_contiguous()
                and v.is_contiguous() and k.dtype == torch.bfloat16 and v.dtype == torch.bfloat16):
            raise ValueError("q, k, v must be contiguous bf16 CUDA tensors")
        if q.shape != (plan.total_q, plan.num_q_heads, plan.head_dim) or \
                k.shape != (plan.total_k, plan.num_kv_heads, plan.head_dim) or v.shape != k.shape:
            raise ValueError("tensor shapes do not match the plan")
        o = torch.empty_like(q)
        lse = torch.empty((plan.num_q_heads, plan.total_q), dtype=torch.float32, device=q.device)
        B.skrull_attn_fwd(plan, q, k, v, o, lse)
        ctx.plan = plan
        ctx.save_for_backward(q, k, v, o, lse)
        return o

    @staticmethod
    def backward(ctx, d_o):
        q, k, v, o, lse = ctx.saved_tensors
        plan = ctx.plan
        d_o = d_o.contiguous()
        dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
        ws = torch.empty(max(int(plan.bwd_workspace_bytes), 16), dtype=torch.uint8, device=q.device)
        B.skrull_attn_bwd(plan, q, k, v, o, lse, d_o, dq, dk, dv, ws)
        return dq, dk, dv, None


def _watched():
    """Whether something follows torch's calls from Python (a trace, a functorch transform, forward-mode
    gradients, a mode, a compiler), which has to see the Function above."""
    try:
        return (torch._C._get_tracing_state() is not None or torch._C._functorch.peek_interpreter_stack() is not None
                or torch.autograd.forward_ad._current_level >= 0 or torch._C._len_torch_dispatch_stack() > 0
                or torch._C._len_torch_function_stack() > 0 or torch.compiler.is_compiling())
    except AttributeError:   # (most of these are private to torch)
        return True


_native = None   # the same in native code; False where that cannot be loaded


def _load_native():
    """csrc/autograd.cpp, built in-tree with the library against the torch of that build.  The library's kernels are called either
    way: without this module, or with one for another torch, by the Function above."""
    global _native
    B.lib()
    try:
        from . import _autograd
    except ImportError as e:
        warnings.warn(f"paper_2505_19609_amd/_autograd.so cannot be loaded ({e}): calls of skrull_attention take the host "
                      "longer; build it with python -m paper_2505_19609_amd.build", RuntimeWarning, stacklevel=3)
        _native = False
    else:
        _autograd.set_check(B._check)
        _native = _autograd.attention
    return _native


_TENSORS = (torch.Tensor, torch.nn.Parameter)


def skrull_attention(q, k, v, plan):
    """O = packed varlen causal attention of the micro-batch `plan` describes
    (a binding.Plan); differentiable with respect to q, k, v."""
    if type(q) in _TENSORS and type(k) in _TENSORS and type(v) in _TENSORS and type(plan) is B.Plan and not _watched():
        native = _load_native() if _native is None else _native
        if native:
            i = plan.info
            return native(q, k, v, plan, i.total_q, i.total_k, i.num_q_heads, i.num_kv_heads, i.head_dim)
    return _SkrullAttention.apply(q, k, v, plan)
