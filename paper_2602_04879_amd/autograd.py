"""The loss as a torch.autograd.Function, for a trainer that wants `loss.backward()`.

Argument marshalling only.  The library computes the loss and its gradient with respect to the
logits in ONE pass (dppo_loss_fwd_bwd of include/dppo.h: Eq. dppo_obj for the loss, Eq.
unified_grad for the gradient, the mask a constant), so `forward` already holds the gradient and
`backward` only hands it over, scaled by the incoming gradient of the scalar loss.  There is no
CPU fallback: without the HIP library the call raises.

    loss, aux = dppo_loss(logits, sampled_ids, mu_logp, advantages, delta=0.2, variant=BINARY_TV,
                          loss_scale=1.0 / T)
    loss.backward()            # logits.grad (bf16) is the fused kernel's gradient

`aux` holds the per-token divergence, mask and loss terms (no gradient flows through them).
With `in_place=True` the gradient is written over the logits' own storage (allowed by the
boundary): the logits are then consumed by the call, as a fused cross-entropy would consume them.
"""
from __future__ import annotations

import torch
import torch.autograd.forward_ad as fwAD

from . import binding as B


# Gradients of this many entries and more are scaled by a kernel that reads the incoming gradient of the
# loss on the device; smaller ones look at it on the host and are left alone if it is one.  Looking is a
# synchronisation, behind which the device idles while the host prepares the next call (4096 x 256000: 886 us a step,
# 819 without); but the library call from autograd's own thread costs the host about 25 us more than the look (256 x 4096, plain
# backward: 130 us a step against 106), which counts as long as the device's own work is shorter than the host's.  A step of the
# logits' loss, factor one, looked at / read by the kernel: 2^26 entries 119-128 / 140 us, 1400 x 50257 (1.05 x 2^26) 131 / 144, 2^27
# entries 173-189 / 141.  (The hidden-state loss goes by its larger gradient: its products alone take longer than either.)
SCALE_ON_DEVICE_FROM = 5 << 24

# What a pending hidden-state loss may hold beyond the 4 V d bytes of the weight's gradient in fp32 to have that gradient formed in
# backward: an eighth of them (the logits' gradient is as large as they are at T = 2 d), or this, a thousandth of the card's memory.  A step
# that sums the losses of several micro-batches before one backward holds every one of them: 8192 tokens x 768 at V = 151936 would
# be 2.5 GB each in place of 0.47.  Formed in fp32 in forward, such a step takes 1.03-1.04 of the time at 8192 x 768 .. 3584, 1.05-1.06 at 4096 x
# 768 and 1024; what this lets pass would take 1.09 at 2048 x 768 and, V = 32768, 1.17 at 3000 x 1024 (597 / 700 us), V = 16000, 1.07 at 8192 x 2048.
HELD_MORE = 256 << 20


def _grad_like(logits: torch.Tensor) -> torch.Tensor:
    """An empty gradient for rows of `logits`, with the same row pitch: the boundary has one pitch for
    both.  (torch.empty_like drops the pitch of a slice logits[:, :V] and returns packed rows.)"""
    if logits.is_contiguous():
        return torch.empty_like(logits)
    T, V = logits.shape
    ld = logits.stride(0) if T > 1 else V
    return logits.new_empty((T, max(ld, V)))[:, :V]


class _DppoLoss(torch.autograd.Function):
    @staticmethod
    def forward(ctx, logits, sampled_ids, mu_logp, advantages, mu_topk_ids, mu_topk_logp, mu_logits, opts):
        if logits.dtype != torch.bfloat16 or logits.dim() != 2 or not logits.is_cuda:
            raise ValueError("logits: a bf16 [T, V] tensor on the GPU")
        if logits.stride(1) != 1:
            raise ValueError("logits: rows must be contiguous")
        T = logits.shape[0]
        out = B.alloc_outputs(T, logits.device, want_diagnostics=opts.get("diagnostics", False))
        need_grad = ctx.needs_input_grad[0]
        grad = None
        if need_grad:
            grad = logits.detach() if opts.get("in_place", False) else _grad_like(logits)
        args = B.make_args(logits.detach(), sampled_ids, mu_logp, advantages, opts["delta"], opts["variant"], opts["loss_scale"], out,
                           mu_topk_ids, mu_topk_logp, grad_logits=grad, mu_logits=mu_logits,
                           mask_rule=opts.get("mask_rule", B.MASK_DIVERGENCE), eps_low=opts.get("eps_low", 0.2),
                           eps_high=opts.get("eps_high", 0.2), ratio_cap=opts.get("ratio_cap", 0.0), flags=opts.get("flags", 0),
                           anchor_logp=opts.get("anchor_logp"), relax_alpha=opts.get("relax_alpha", 0.0),
                           relax_sides=opts.get("relax_sides", 0))
        (B.dppo_loss_fwd_bwd if need_grad else B.dppo_loss_fwd)(args)
        ctx.grad_logits, ctx.own_buffer = grad, not opts.get("in_place", False)
        side = [out[k] for k in ("divergence", "mask", "loss_tok")] + ([out["diagnostics"]] if out["diagnostics"] is not None else [])
        ctx.mark_non_differentiable(*side)
        return (out["loss"].reshape(()), *side)

    @staticmethod
    def backward(ctx, grad_loss, *unused):
        g = ctx.grad_logits
        ctx.grad_logits = None
        if g is None:
            return (None,) * 8
        # d(out)/d(logits) = grad_loss * d(loss)/d(logits); the scale is applied in fp32 and rounded once
        if ctx.own_buffer and g.numel() >= SCALE_ON_DEVICE_FROM and _value_only(grad_loss):
            g = B.scale_rows_(g, _in_memory(grad_loss))
        elif not _is_one(grad_loss):
            # known on the host by now: one multiplication where the gradient lies (as three tensor operations over
            # fp32 copies: 600 x 50257 rows at a pitch of 50304, loss / 4, 172 us a step, 146 now)
            if ctx.own_buffer and _value_only(grad_loss):
                g = g.mul_(float(grad_loss))
            else:       # a derivative through grad_loss is wanted, or the gradient is in the logits' own storage, which stays as it is
                g = (g.float() * grad_loss.float()).to(torch.bfloat16)
        return (g, None, None, None, None, None, None, None)


def _value_only(grad_loss: torch.Tensor) -> bool:
    """Whether the result is wanted as a value and not as a function of grad_loss: no graph through it
    (create_graph) and no tangent on it (forward mode over this backward).  A kernel keeps neither."""
    return not torch.is_grad_enabled() and fwAD.unpack_dual(grad_loss).tangent is None


def _in_memory(grad_loss: torch.Tensor) -> torch.Tensor:
    """grad_loss with its value in memory, where a kernel reads it: an engine also hands over lazily negated
    views (z.conj().imag as the incoming gradient, or from a hook on the loss) and zeros without memory."""
    grad_loss = grad_loss.resolve_neg()
    return grad_loss if grad_loss.data_ptr() else grad_loss.clone()


def _is_one(t: torch.Tensor) -> bool:
    # a scalar one, known on the host only at the cost of a synchronisation, which one scalar read is
    return t.numel() == 1 and float(t) == 1.0


def dppo_loss(logits, sampled_ids, mu_logp, advantages, *, delta, variant=B.BINARY_TV, loss_scale=1.0,
              mu_topk_ids=None, mu_topk_logp=None, mu_logits=None, **opts):
    """loss (a 0-d fp32 tensor with a gradient path to `logits`) and a dict of the per-token
    outputs.  Keyword options: mask_rule, eps_low, eps_high, ratio_cap (the baselines of the
    unified gradient form), anchor_logp (the mask anchored to a recomputed policy: MiniRL, the
    decoupled objective), relax_alpha / relax_sides (the clip relaxed for low-probability tokens),
    diagnostics, in_place, flags."""
    opts = dict(opts, delta=float(delta), variant=int(variant), loss_scale=float(loss_scale))
    res = _DppoLoss.apply(logits, sampled_ids, mu_logp, advantages, mu_topk_ids, mu_topk_logp, mu_logits, opts)
    aux = {"divergence": res[1], "mask": res[2], "loss_tok": res[3]}
    if len(res) > 4:
        aux["diagnostics"] = res[4]
    return res[0], aux


class _DppoLmheadLoss(torch.autograd.Function):
    @staticmethod
    def forward(ctx, hidden, weight, sampled_ids, mu_logp, advantages, mu_topk_ids, mu_topk_logp, opts):
        if hidden.dtype != torch.bfloat16 or weight.dtype != torch.bfloat16 or hidden.dim() != 2 or weight.dim() != 2:
            raise ValueError("hidden [T, d] and weight [V, d]: bf16 matrices on the GPU")
        if hidden.stride(1) != 1 or weight.stride(1) != 1 or hidden.shape[1] != weight.shape[1]:
            raise ValueError("hidden and weight: contiguous rows of the same length d")
        T, d = hidden.shape
        V = weight.shape[0]
        need_h, need_w = ctx.needs_input_grad[0], ctx.needs_input_grad[1]
        backward = need_h or need_w
        batch = {"hidden": hidden.detach(), "weight": weight.detach(), "d": d, "V": V, "sampled_ids": sampled_ids, "mu_logp": mu_logp,
                 "advantages": advantages, "delta": opts["delta"], "variant": opts["variant"], "loss_scale": opts["loss_scale"],
                 "mu_topk_ids": mu_topk_ids, "mu_topk_logp": mu_topk_logp, "anchor_logp": opts.get("anchor_logp")}
        chunk = opts.get("chunk_rows", 0)
        # One chunk: the logits' gradient stays as it is in the workspace, and the weight's gradient is formed from it in
        # backward, where its factor is known, straight in the weight's type (V = 151936, d = 2048, 1000 tokens: 2158 us a step,
        # 1775 now; 64 tokens x 768: 416 / 283).  Several chunks are summed in fp32; so is one of more rows than a chunk has
        # unasked.  And so are tokens whose logits' gradient would be far more to hold than the weight's in fp32: see HELD_MORE.
        later = need_w and 0 < T <= min(chunk if chunk > 0 else T, B.LMHEAD_CHUNK_ROWS)
        if later:
            room = B.lmhead_workspace_bytes(T, V, chunk)
            later = room + 2 * T * d <= 4 * V * d + max(V * d // 2, HELD_MORE)
        # (no tokens: the library runs no product and leaves the buffer as it is)
        gw = (torch.empty if T > 0 else torch.zeros)((V, d), dtype=torch.float32, device=hidden.device) if need_w and not later else None
        rule = {k: opts[k] for k in ("mask_rule", "eps_low", "eps_high", "ratio_cap", "relax_alpha", "relax_sides") if k in opts}
        # what is kept lies in a workspace of its own, without the room for the divided contraction (up to 1 GiB) behind it
        workspace, scratch = B.alloc_lmhead_apart(T, V, d, chunk, hidden.device, room) if later else (None, None)
        res = B.run_lmhead(batch, backward=backward, chunk_rows=chunk, diagnostics=opts.get("diagnostics", False),
                           grad_weight=gw, flags=opts.get("flags", 0), workspace=workspace, scratch=scratch, **rule)
        # (a copy of the hidden states: the caller may write to its own before backward)
        ctx.factors = (B.lmhead_logit_gradients(res["workspace_buf"], T, V), hidden.detach().clone(memory_format=torch.contiguous_format)) if later else None
        ctx.grads = (res["grad_hidden"] if need_h else None, gw)
        side = [res[k] for k in ("divergence", "mask", "loss_tok")] + ([res["diagnostics"]] if res["diagnostics"] is not None else [])
        ctx.mark_non_differentiable(*side)
        return (res["loss"].reshape(()), *side)

    @staticmethod
    def backward(ctx, grad_loss, *unused):
        gh, gw = ctx.grads
        factors = ctx.factors
        ctx.grads = ctx.factors = None
        if factors is not None:
            if _value_only(grad_loss):
                grad_loss = _in_memory(grad_loss)
                gw = B.gemm_tn_bf16(*factors, grad_loss)
                if gh is not None:
                    gh = B.scale_rows_(gh, grad_loss)
                return (gh, gw, None, None, None, None, None, None)
            g, h = factors
            gw = B.gemm_tn_f32(g, h, torch.empty((g.shape[1], h.shape[1]), dtype=torch.float32, device=g.device))
        big = max(t.numel() if t is not None else 0 for t in (gh, gw)) >= SCALE_ON_DEVICE_FROM
        if big and _value_only(grad_loss):
            grad_loss = _in_memory(grad_loss)
            if gh is not None:
                gh = B.scale_rows_(gh, grad_loss)
            if gw is not None:      # accumulated in fp32; autograd wants the weight's own type
                gw = B.scale_to_bf16(gw, grad_loss)
            return (gh, gw, None, None, None, None, None, None)
        one = _is_one(grad_loss)
        if gh is not None and not one:
            gh = (gh.float() * grad_loss.float()).to(torch.bfloat16)
        if gw is not None:
            gw = (gw if one else gw * grad_loss.float()).to(torch.bfloat16)
        return (gh, gw, None, None, None, None, None, None)


def dppo_lmhead_loss(hidden, weight, sampled_ids, mu_logp, advantages, *, delta, variant=B.BINARY_TV, loss_scale=1.0,
                     mu_topk_ids=None, mu_topk_logp=None, **opts):
    """The same loss one step earlier (dppo_lmhead_loss_fwd[_bwd] of include/dppo.h): from the final
    hidden states [T, d] and the lm_head weight [V, d], both bf16; the logits exist a chunk of
    tokens at a time inside the call (forward only: never).  Returns the loss, with gradient paths
    to `hidden` and `weight`, and the per-token outputs.  Options as for dppo_loss, plus chunk_rows."""
    opts = dict(opts, delta=float(delta), variant=int(variant), loss_scale=float(loss_scale))
    res = _DppoLmheadLoss.apply(hidden, weight, sampled_ids, mu_logp, advantages, mu_topk_ids, mu_topk_logp, opts)
    aux = {"divergence": res[1], "mask": res[2], "loss_tok": res[3]}
    if len(res) > 4:
        aux["diagnostics"] = res[4]
    return res[0], aux
