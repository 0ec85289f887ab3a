"""torch.autograd wrapper over the C-ABI calls of binding.py (fine-tuning use of Section 5).

    O = sla_attention(Q, K, V, W, k_h=0.05, k_l=0.10)

runs sla_build_mask + sla_forward and records sla_backward; every step is a kernel of
libsla_hip.so, this module only keeps the buffers alive between the two passes.  The mask is a
constant of the graph (no gradient flows into the block scores); a mask built once can be passed
back in through `mask=` and reused, e.g. across the steps of a diffusion sampler.
"""
from __future__ import annotations

from typing import Optional, Tuple

import torch

from . import binding as sla


class _SLAFunction(torch.autograd.Function):
    @staticmethod
    def forward(ctx, Q, K, V, W, p, Mc, luts, grad):
        # the library reads W in the storage type of Q, K, V (a float parameter next to bf16
        # activations is cast here; its gradient goes back in the parameter's own type)
        ctx.w_dtype = W.dtype
        W = W.detach()
        if W.dtype != Q.dtype or not W.is_contiguous():
            W = W.to(Q.dtype).contiguous()
        # without a backward pass to come (grad false) O^s, O^l, L stay on the chip and H, Z in the
        # workspace: two thirds of the forward kernel's stores (16 x 16 heads x 1024 tokens, d = 64: 53 -> 46 us)
        if Mc is None:
            Mc, luts, O, saved = sla.sla_mask_forward(p, Q, K, V, W, need_saved=grad)
        else:
            O, saved = sla.sla_forward(p, Q, K, V, W, Mc, luts, need_saved=grad)
        if grad:
            ctx.p = p
            ctx.save_for_backward(Q, K, V, W, Mc, luts, saved)
        return O

    @staticmethod
    def backward(ctx, dO):
        Q, K, V, W, Mc, luts, saved = ctx.saved_tensors
        dt = torch.bfloat16 if ctx.w_dtype == torch.bfloat16 else torch.float32
        dQ, dK, dV, dW = sla._backward(ctx.p, Q, K, V, W, Mc, luts, saved, dO.contiguous(), None, None, dt)
        return dQ, dK, dV, dW.to(ctx.w_dtype), None, None, None, None


def _params(Q, k_h, k_l, phi, token_major, bq) -> sla.sla_params:
    if token_major:
        B, N, H, d = Q.shape
    else:
        B, H, N, d = Q.shape
    return sla.make_params(B, H, N, d, k_h, k_l, Q.dtype, phi=phi, bq=bq,
                           layout=sla.SLA_BNHD if token_major else sla.SLA_BHND)


def build_mask(Q: torch.Tensor, K: torch.Tensor, k_h: float, k_l: float,
               phi: int = sla.SLA_PHI_SOFTMAX, token_major: bool = False, bq: int = 64
               ) -> Tuple[sla.sla_params, torch.Tensor, torch.Tensor]:
    """(params, M_c int8 [B,H,ceil(N/bq),ceil(N/64)], lookup tables) for contiguous [B,H,N,d]
    tensors, or [B,N,H,d] ones with token_major.  bq: query block size of the mask (64 .. 256)."""
    p = _params(Q, k_h, k_l, phi, token_major, bq)
    Mc, luts, _ = sla.sla_build_mask(p, Q, K)   # (only the tensors' memory is handed on: no part of a graph)
    return p, Mc, luts


def sla_attention(Q: torch.Tensor, K: torch.Tensor, V: torch.Tensor, W: torch.Tensor,
                  k_h: float = 0.05, k_l: float = 0.10, phi: int = sla.SLA_PHI_SOFTMAX,
                  mask: Optional[Tuple[sla.sla_params, torch.Tensor, torch.Tensor]] = None,
                  token_major: bool = False, bq: int = 64) -> torch.Tensor:
    """O = O^s + Proj(O^l) (Eq. 6) with gradients to Q, K, V and the Proj weight W [d, d].
    Q, K, V (and O, and the gradients) are [B,H,N,d], or [B,N,H,d] with token_major -- the order
    in which a transformer block's projections leave them, no transpose needed."""
    p, Mc, luts = mask if mask is not None else (_params(Q, k_h, k_l, phi, token_major, bq), None, None)
    grad = torch.is_grad_enabled() and any(
        getattr(t, "requires_grad", False) for t in (Q, K, V, W))
    return _SLAFunction.apply(Q, K, V, W, p, Mc, luts, grad)
