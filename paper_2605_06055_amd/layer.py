"""Device buffers of one MoE layer's dispatch/combine plus the three calls in order.

Memory plumbing only: torch allocates the tensors and provides the stream; every step of the
path runs in the HIP library through the binding.
"""
from __future__ import annotations

import numpy as np

from . import binding as B


def to_device(a: np.ndarray, device="cuda"):
    """numpy -> torch on the GPU; uint16 arrays are bf16 bit patterns."""
    import torch
    if a.dtype == np.uint16:
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).to(device).view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(a)).to(device)


def to_host(t) -> np.ndarray:
    import torch
    if t.dtype == torch.bfloat16:
        return t.view(torch.int16).cpu().numpy().view(np.uint16)
    return t.cpu().numpy()


class MoeLayer:
    """Buffers for shape (T,H,k,E,R): plan state, window, expert_out, Y."""

    def __init__(self, T, H, k, E, R, dtype=B.MOE_DTYPE_BF16, schedule=B.MOE_SCHEDULE_AUTO,
                 region_stride_rows=0, device="cuda", separate_expert_out=True, source_count=None, rank_id=0,
                 window_rows=None):
        import torch
        self.shape = B.MoeShape(T=T, H=H, k=k, E=E, R=R, dtype=dtype, schedule=schedule, rank_id=rank_id,
                                region_stride_rows=region_stride_rows)
        self.torch_dtype = torch.bfloat16 if dtype == B.MOE_DTYPE_BF16 else torch.float32
        # with several source ranks the caller, who holds the count matrix, sizes tight windows
        self.rows = B.moe_window_rows(self.shape) if window_rows is None else window_rows
        self.schedule = B.moe_resolve_schedule(self.shape)
        self.plan = B.MoePlan(self.shape, device=device, source_count=source_count)
        self._plan_struct = self.plan.struct()
        self.prefetch_x = False
        self.window = torch.empty((max(self.rows, 1), H), dtype=self.torch_dtype, device=device)
        self.expert_out = (torch.empty_like(self.window) if separate_expert_out else self.window)
        self.y = torch.empty((max(T, 1), H), dtype=self.torch_dtype, device=device)

    def dispatch(self, x, topk_idx, stream=None):
        """Plan (prefill schedule only) + dispatch.  With ``prefetch_x`` set the plan is told to pull x into the
        caches while it runs (moe_plan_t.prefetch)."""
        if self.schedule == B.MOE_SCHEDULE_PREFILL:
            if self.prefetch_x:
                plan = self._plan_struct
                plan.prefetch, plan.prefetch_bytes = B._ptr(x), x.numel() * x.element_size()
                try:
                    B.moe_plan(self.shape, topk_idx, plan, stream)
                finally:                      # the structure outlives x
                    plan.prefetch, plan.prefetch_bytes = None, 0
            else:
                B.moe_plan(self.shape, topk_idx, self._plan_struct, stream)
        B.moe_dispatch(self.shape, x, topk_idx, self._plan_struct, self.window, stream)

    def combine(self, topk_w, stream=None):
        B.moe_combine(self.shape, self.expert_out, topk_w, self._plan_struct, self.y, stream)

    def bind(self, x, topk_idx, topk_w, stream=None):
        """Pre-marshalled calls for a serving loop that re-runs the layer on the same buffers: returns
        (dispatch, combine) callables whose arguments were read once.  The stream is the one
        current at bind time unless given.  Each of the two keeps the buffers alive, without the layer too."""
        st = B._stream(stream) or 0
        tensors = (x, topk_idx, topk_w, self.window, self.expert_out, self.y)
        return B._bind(self.shape, self._plan_struct, self.schedule == B.MOE_SCHEDULE_PREFILL, *(B._ptr(t) for t in tensors), st,
                       (tensors, tuple(vars(self.plan).values())))
