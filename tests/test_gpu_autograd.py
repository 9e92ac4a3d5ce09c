"""The torch.autograd wrapper of the loss: loss.backward() must deliver the fused kernel's gradient
(argument marshalling only: compared with the oracle like every other GPU result)."""
import numpy as np
import pytest
import torch
import torch.autograd.forward_ad as fwAD

from paper_2602_04879_amd import autograd as A
from paper_2602_04879_amd import binding as B
from paper_2602_04879_amd import workloads as W
from tests import parity as P

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _call(b, logits, **kw):
    K = b["K"]
    return A.dppo_loss(logits, b["sampled_ids"], b["mu_logp"], b["advantages"], delta=b["delta"], variant=b["variant"],
                       loss_scale=b["loss_scale"], mu_topk_ids=b["mu_topk_ids"] if K else None,
                       mu_topk_logp=b["mu_topk_logp"] if K else None, **kw)


@pytest.mark.parametrize("variant,K,V", [(W.BINARY_TV, 0, 4096), (W.TOPK_KL, 20, 16384), (W.BINARY_KL, 0, 3001)])
def test_backward_delivers_the_fused_gradient(variant, K, V):
    w = W.Workload("autograd", 3, 40, V, variant, 0.05 if variant in (W.BINARY_KL, W.TOPK_KL) else 0.2, K=K,
                   logit_std=3.0, noise_std=1.0, adv="normal", seed=91)
    b = W.make_batch(w, DEV, shift_sampled=2.0)
    print(f"[case] autograd variant={variant} K={K} V={V} T={b['T']}", flush=True)
    rows = np.arange(b["T"])
    ref = P.oracle_rows(b, rows)
    logits = b["logits"].clone().requires_grad_(True)
    loss, aux = _call(b, logits, diagnostics=True)
    assert loss.requires_grad and not aux["divergence"].requires_grad
    loss.backward()
    torch.cuda.synchronize()
    res = dict(aux, loss=loss.detach().reshape(1), grad_logits=logits.grad)
    st = P.compare_rows(b, res, rows, ref=ref)
    P.check_loss_scalar(b, res, float(ref["loss_tok"].sum()))
    assert 0 < st["masked"] < b["T"]
    # the gradient of 3 * loss is 3 * the gradient, rounded once more to bf16
    logits3 = b["logits"].clone().requires_grad_(True)
    loss3, _ = _call(b, logits3)
    (3.0 * loss3).backward()
    torch.cuda.synchronize()
    want = (logits.grad.float() * 3.0).to(torch.bfloat16)
    assert torch.equal(logits3.grad, want)
    # without a gradient path the forward-only entry point runs and nothing is allocated for a gradient
    with torch.no_grad():
        loss0, aux0 = _call(b, b["logits"])
    torch.cuda.synchronize()
    assert not loss0.requires_grad
    assert torch.equal(aux0["divergence"], aux["divergence"]) and torch.equal(aux0["mask"], aux["mask"])
    assert abs(loss0.item() - loss.item()) <= 1e-6 * abs(loss.item()) + 1e-12


def test_in_place_gradient_over_the_logits():
    w = W.Workload("autograd_inplace", 2, 64, 16384, W.TOPK_TV, 0.1, K=8, logit_std=3.0, noise_std=1.0, adv="normal", seed=93)
    b = W.make_batch(w, DEV, shift_sampled=2.0)
    keep = b["logits"].clone().requires_grad_(True)
    loss_ref, _ = _call(b, keep)
    loss_ref.backward()
    leaf = b["logits"].clone().requires_grad_(True)
    storage = leaf.data_ptr()
    loss, _ = _call(b, leaf, in_place=True)
    loss.backward()
    torch.cuda.synchronize()
    assert torch.equal(leaf.grad, keep.grad) and torch.equal(loss.detach(), loss_ref.detach())
    assert leaf.grad.data_ptr() == storage          # the gradient lives in the logits' own storage


def test_hidden_state_form_backward_matches_the_direct_call():
    w = W.Workload("autograd_lm", 2, 150, 4160, W.TOPK_TV, 0.1, K=8, logit_std=3.0, noise_std=1.0, adv="normal", seed=95)
    b = W.make_lmhead_batch(w, 128, DEV, exact=True, shift_sampled=2.0)
    gw_ref = torch.empty((b["V"], b["d"]), dtype=torch.float32, device=DEV)
    ref = B.run_lmhead(b, chunk_rows=64, grad_weight=gw_ref)
    h = b["hidden"].clone().requires_grad_(True)
    wt = b["weight"].clone().requires_grad_(True)
    loss, aux = A.dppo_lmhead_loss(h, wt, b["sampled_ids"], b["mu_logp"], b["advantages"], delta=b["delta"], variant=b["variant"],
                                   loss_scale=b["loss_scale"], mu_topk_ids=b["mu_topk_ids"], mu_topk_logp=b["mu_topk_logp"], chunk_rows=64)
    loss.backward()
    torch.cuda.synchronize()
    assert torch.equal(loss.detach().reshape(1), ref["loss"]) and torch.equal(aux["mask"], ref["mask"])
    assert torch.equal(aux["divergence"], ref["divergence"])
    assert torch.equal(h.grad, ref["grad_hidden"])
    assert torch.equal(wt.grad, gw_ref.to(torch.bfloat16))
    assert 0 < (aux["mask"] == 0).sum().item() < b["T"]
    # forward only (no gradient path): no logit is written, same per-token results up to summation order
    with torch.no_grad():
        loss0, aux0 = A.dppo_lmhead_loss(b["hidden"], b["weight"], b["sampled_ids"], b["mu_logp"], b["advantages"], delta=b["delta"],
                                         variant=b["variant"], loss_scale=b["loss_scale"], mu_topk_ids=b["mu_topk_ids"],
                                         mu_topk_logp=b["mu_topk_logp"], chunk_rows=64)
    torch.cuda.synchronize()
    assert B.last_path() == "lmhead_fused"
    assert torch.equal(aux0["mask"], ref["mask"])
    assert torch.allclose(aux0["divergence"], ref["divergence"], rtol=1e-4, atol=1e-7)


@pytest.mark.parametrize("V,ld", [(4090, 4096), (3001, 3072), (50257, 50304)])
def test_backward_of_a_slice_of_padded_logits(V, ld):
    """logits[:, :V] of a padded buffer: the gradient has the buffer's pitch, its values are those of the
    direct call, and the bytes around it stay as they were."""
    w = W.Workload("autograd_pitch", 2, 37, V, W.BINARY_TV, 0.2, logit_std=3.0, noise_std=1.0, adv="normal", seed=97)
    b = W.make_batch(w, DEV, ld=ld, shift_sampled=2.0)
    print(f"[case] autograd pitch V={V} ld={ld}", flush=True)
    direct = torch.full_like(b["logits"], 7.0)
    B.run_batch(b, grad=direct)
    logits = b["logits"][:, :V].detach().requires_grad_(True)
    loss, _ = _call(b, logits)
    g, = torch.autograd.grad(loss, logits)
    torch.cuda.synchronize()
    assert g.stride() == logits.stride() and torch.equal(g, direct[:, :V])
    assert (direct[:, V:] == 7.0).all()


@pytest.mark.parametrize("rows,cols,ld,off", [(1, 1, 1, 0), (1, 7, 7, 3), (3, 8, 8, 0), (5, 8189, 8192, 1), (4, 8193, 8193, 0),
                                              (2, 65537, 65544, 5), (300, 4099, 4099, 7), (3000, 1024, 1088, 0)])
def test_scaled_gradient_rows(rows, cols, ld, off):
    """x *= factor over rows of any pitch and alignment: the fp32 product rounded once, the entries
    around the rows untouched, and a factor of one leaving every bit alone."""
    g = torch.Generator(device=DEV); g.manual_seed(rows + cols)
    buf = torch.randn(off + rows * ld + 9, generator=g, device=DEV).to(torch.bfloat16)
    buf[off] = float("inf")
    keep = buf.clone()
    x = buf[off:off + rows * ld].view(rows, ld)[:, :cols]
    print(f"[case] scale rows={rows} cols={cols} ld={ld} off={off}", flush=True)
    B.scale_rows_(x, torch.ones((), device=DEV))
    torch.cuda.synchronize()
    assert torch.equal(buf, keep)
    f = torch.tensor(-0.3125 / 3, device=DEV)
    B.scale_rows_(x, f)
    torch.cuda.synchronize()
    want = keep.clone()
    v = want[off:off + rows * ld].view(rows, ld)[:, :cols]
    v.copy_((v.float() * f).to(torch.bfloat16))
    assert torch.equal(buf, want)
    src = torch.randn(rows * cols, generator=g, device=DEV)
    got = B.scale_to_bf16(src, f)
    torch.cuda.synchronize()
    assert torch.equal(got, (src * f).to(torch.bfloat16))


@pytest.mark.parametrize("chunk_rows,factor", [(0, 1.0), (0, -0.3), (80, -0.3), (79, -0.3)])
def test_weight_gradient_formed_in_backward_is_that_of_the_direct_call(chunk_rows, factor):
    """One chunk: the weight's gradient is formed in backward, from what forward saw (the hidden states are
    overwritten in between); its bits are those of the fp32 gradient scaled and rounded once."""
    b = W.make_lmhead_batch(W.Workload("autograd_later", 2, 40, 4160, W.BINARY_TV, 0.2, logit_std=3.0, noise_std=1.0, adv="normal", seed=113), 192, DEV)
    f = torch.tensor(factor, device=DEV)
    gw = torch.empty((b["V"], b["d"]), dtype=torch.float32, device=DEV)
    ref = B.run_lmhead(b, grad_weight=gw, chunk_rows=chunk_rows)
    h, wt = b["hidden"].clone().requires_grad_(True), b["weight"].clone().requires_grad_(True)
    loss, _ = A.dppo_lmhead_loss(h, wt, b["sampled_ids"], b["mu_logp"], b["advantages"], delta=b["delta"], variant=b["variant"],
                                 loss_scale=b["loss_scale"], chunk_rows=chunk_rows)
    with torch.no_grad():
        h.fill_(7.0)
    gh, g = torch.autograd.grad(loss, (h, wt), f)
    torch.cuda.synchronize()
    assert torch.equal(g, (gw * f).to(torch.bfloat16)) and torch.equal(gh, (ref["grad_hidden"].float() * f).to(torch.bfloat16))


@pytest.mark.parametrize("entries", [0, 1 << 40])
@pytest.mark.parametrize("chunk_rows", [0, 64])
def test_no_tokens_give_zero_gradients(monkeypatch, chunk_rows, entries):
    """T = 0: no product runs, and the weight's gradient is zero whatever its memory held before (blocks of its size, in
    both types, are freed full of NaN first)."""
    monkeypatch.setattr(A, "SCALE_ON_DEVICE_FROM", entries)
    b = W.make_lmhead_batch(W.Workload("autograd_empty", 1, 4, 4160, W.BINARY_TV, 0.2, logit_std=3.0, noise_std=1.0, adv="normal", seed=115), 192, DEV)
    wt = b["weight"].clone().requires_grad_(True)
    for factor in (1.0, 0.3):
        h = b["hidden"][:0].clone().requires_grad_(True)
        blocks = [torch.full((b["V"], b["d"]), float("nan"), dtype=dt, device=DEV) for dt in (torch.float32, torch.bfloat16) for _ in range(3)]
        del blocks
        loss, _ = A.dppo_lmhead_loss(h, wt, b["sampled_ids"][:0], b["mu_logp"][:0], b["advantages"][:0], delta=b["delta"], variant=b["variant"],
                                     loss_scale=b["loss_scale"], chunk_rows=chunk_rows)
        gh, gw = torch.autograd.grad(loss * factor, (h, wt))
        torch.cuda.synchronize()
        assert loss.item() == 0.0 and gh.shape == h.shape and gw.shape == wt.shape and gw.dtype == wt.dtype
        assert (gw == 0).all()


def test_gradient_with_a_graph_through_the_incoming_gradient():
    """create_graph keeps the path from the gradient to the weight of the loss."""
    w = W.Workload("autograd_graph", 2, 16, 4096, W.BINARY_TV, 0.5, logit_std=3.0, noise_std=0.3, adv="normal", seed=99)
    b = W.make_batch(w, DEV)
    logits = b["logits"].clone().requires_grad_(True)
    u = torch.tensor(0.5, device=DEV, requires_grad=True)
    loss, _ = _call(b, logits)
    g, = torch.autograd.grad(loss * u, logits, create_graph=True)
    du, = torch.autograd.grad(g.float().square().sum(), u)
    plain = b["logits"].clone().requires_grad_(True)
    loss1, _ = _call(b, plain)
    loss1.backward()
    torch.cuda.synchronize()
    want = plain.grad.double().square().sum().item()          # d/du sum (u g)^2 = 2 u sum g^2, u = 1/2: exact in bf16
    assert abs(du.item() - want) <= 1e-2 * want


@pytest.mark.parametrize("chunk_rows", [0, 32])
@pytest.mark.parametrize("factor", [1.0, 0.3])
def test_scaling_on_the_device_and_on_the_host_give_the_same_gradients(monkeypatch, factor, chunk_rows):
    """Large gradients are scaled by a kernel that reads the factor, small ones by tensor operations
    behind a look at it: the same bits (here on one small call each way).  Of the hidden states, the weight's gradient is left to
    scale where several chunks were summed in fp32; one chunk's is formed with the factor, whatever its size."""
    w = W.Workload("autograd_scale", 2, 40, 8192, W.BINARY_TV, 0.2, logit_std=3.0, noise_std=1.0, adv="normal", seed=103)
    b = W.make_batch(w, DEV, shift_sampled=2.0)
    lb = W.make_lmhead_batch(W.Workload("autograd_scale_lm", 2, 40, 4160, W.BINARY_TV, 0.2, logit_std=3.0, noise_std=1.0, adv="normal", seed=105), 64, DEV)
    got, conversions, convert = [], [], B.scale_to_bf16
    monkeypatch.setattr(B, "scale_to_bf16", lambda *a: conversions.append(1) or convert(*a))
    for entries in (0, 1 << 40):
        monkeypatch.setattr(A, "SCALE_ON_DEVICE_FROM", entries)
        logits = b["logits"].clone().requires_grad_(True)
        loss, _ = _call(b, logits)
        h, wt = lb["hidden"].clone().requires_grad_(True), lb["weight"].clone().requires_grad_(True)
        lloss, _ = A.dppo_lmhead_loss(h, wt, lb["sampled_ids"], lb["mu_logp"], lb["advantages"], delta=lb["delta"], variant=lb["variant"],
                                      loss_scale=lb["loss_scale"], chunk_rows=chunk_rows)
        (factor * loss + factor * lloss).backward()
        torch.cuda.synchronize()
        got.append((logits.grad, h.grad, wt.grad))
        assert len(conversions) == (1 if chunk_rows else 0)         # by the kernel the first time, never the second
    for x, y in zip(*got):
        assert torch.equal(x, y)


def _both_losses(chunk_rows):
    """(inputs, losses of fresh graphs) of one small call of each wrapper, and the plain gradients.  The hidden states in one chunk (0:
    the weight's gradient is formed in backward) or several (summed in fp32)."""
    w = W.Workload("autograd_in", 2, 40, 8192, W.BINARY_TV, 0.2, logit_std=3.0, noise_std=1.0, adv="normal", seed=107)
    b = W.make_batch(w, DEV, shift_sampled=2.0)
    lb = W.make_lmhead_batch(W.Workload("autograd_in_lm", 2, 40, 4160, W.BINARY_TV, 0.2, logit_std=3.0, noise_std=1.0, adv="normal", seed=109), 64, DEV)
    leaves = [b["logits"].clone().requires_grad_(True)], [lb[k].clone().requires_grad_(True) for k in ("hidden", "weight")]

    def losses():
        yield leaves[0], _call(b, leaves[0][0])[0]
        yield leaves[1], A.dppo_lmhead_loss(*leaves[1], lb["sampled_ids"], lb["mu_logp"], lb["advantages"], delta=lb["delta"], variant=lb["variant"],
                                            loss_scale=lb["loss_scale"], chunk_rows=chunk_rows)[0]
    return losses, [torch.autograd.grad(loss, x) for x, loss in losses()]


@pytest.mark.parametrize("chunk_rows", [0, 32])
@pytest.mark.parametrize("entries", [0, 1 << 40])
@pytest.mark.parametrize("how", ["argument", "hook"])
@pytest.mark.parametrize("kind", ["negated", "zero", "plain"])
def test_incoming_gradient_whose_memory_does_not_hold_its_value(monkeypatch, entries, how, kind, chunk_rows):
    """A lazily negated incoming gradient (memory of the opposite sign) and a lazy zero (no memory at all):
    the gradient is that of the value, whichever way it is scaled."""
    monkeypatch.setattr(A, "SCALE_ON_DEVICE_FROM", entries)
    losses, plain = _both_losses(chunk_rows)
    c = {"negated": torch.tensor(0.5 + 0.75j, device=DEV).conj().imag, "zero": torch._efficientzerotensor((), device=DEV),
         "plain": torch.tensor(-0.75, device=DEV)}[kind]
    assert c.is_neg() == (kind == "negated") and (c.data_ptr() == 0) == (kind == "zero")
    value = 0.0 if kind == "zero" else -0.75
    for (x, loss), want in zip(losses(), plain):
        if how == "hook":
            loss.register_hook(lambda g: c)
            got = torch.autograd.grad(loss, x)
        else:
            got = torch.autograd.grad(loss, x, c)
        torch.cuda.synchronize()
        for g, g1 in zip(got, want):
            if value == 0.0:
                assert not g.any()
            else:       # both sides rounded to bf16's 8 significant bits: half a step, 2^-8, each
                assert ((g.float() - value * g1.float()).abs() <= 2.0 ** -7 * g1.float().abs()).all()


@pytest.mark.parametrize("chunk_rows", [0, 32])
@pytest.mark.parametrize("entries", [0, 1 << 40])
def test_tangent_of_the_incoming_gradient(monkeypatch, entries, chunk_rows):
    """Forward mode over the backward: the gradient is linear in the incoming gradient, tangent and all."""
    monkeypatch.setattr(A, "SCALE_ON_DEVICE_FROM", entries)
    losses, plain = _both_losses(chunk_rows)
    for (x, loss), want in zip(losses(), plain):
        with fwAD.dual_level():
            u = fwAD.make_dual(torch.tensor(0.5, device=DEV), torch.tensor(2.0, device=DEV))
            got = [fwAD.unpack_dual(g) for g in torch.autograd.grad(loss, x, u)]
        for g, g1 in zip(got, want):
            # (powers of two: exact)
            assert g.tangent is not None
            assert torch.equal(g.primal, (g1.float() * 0.5).to(torch.bfloat16)) and torch.equal(g.tangent, (g1.float() * 2.0).to(torch.bfloat16))


@pytest.mark.parametrize("V,ld", [(4096, 4096), (4090, 4096), (3001, 3001), (3001, 3072)])
@pytest.mark.parametrize("entries", [0, 1 << 40])
def test_weighted_gradient_stays_in_its_buffer(monkeypatch, V, ld, entries):
    """A factor other than one is applied where the gradient lies, whatever its pitch: no second gradient is
    allocated, and the result is the fp32 product rounded once."""
    monkeypatch.setattr(A, "SCALE_ON_DEVICE_FROM", entries)
    w = W.Workload("autograd_weighted", 2, 37, V, W.BINARY_TV, 0.2, logit_std=3.0, noise_std=1.0, adv="normal", seed=111)
    b = W.make_batch(w, DEV, ld=ld, shift_sampled=2.0)
    logits = b["logits"][:, :V].detach().requires_grad_(True)
    f = torch.tensor(-0.3, device=DEV)                            # fp32, not a bf16 value
    want = (torch.autograd.grad(_call(b, logits)[0], logits)[0].float() * f).to(torch.bfloat16)
    loss, _ = _call(b, logits)
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    g, = torch.autograd.grad(loss, logits, f)
    torch.cuda.synchronize()
    assert torch.cuda.max_memory_allocated() - before < 74 * V and torch.equal(g, want)


@pytest.mark.parametrize("T,V,d,room", [(256, 16384, 768, True), (1536, 16384, 768, True), (300, 8192, 1024, True),
                                        (2048, 16384, 128, False), (4000, 8192, 1024, False), (1700, 16384, 768, False), (1750, 16384, 768, False), (300, 640, 64, False),
                                        (8192, 32768, 64, False)])
@pytest.mark.parametrize("more", [0, None])
def test_memory_held_until_backward(monkeypatch, T, V, d, room, more):
    """Between forward and backward the hidden-state loss holds the logits' gradient, never much more than the weight's in fp32
    would be (`more`: the allowance beside an eighth, None as it is), and none of the scratch that forward alone needed (`room`:
    calls where that would show)."""
    if more is not None:
        monkeypatch.setattr(A, "HELD_MORE", more)
    b = W.make_lmhead_batch(W.Workload("autograd_held", 1, T, V, W.BINARY_TV, 0.2, logit_std=3.0, noise_std=1.0, adv="normal", seed=119), d, DEV)
    h, wt = b["hidden"].requires_grad_(True), b["weight"].requires_grad_(True)

    def forward():
        return A.dppo_lmhead_loss(h, wt, b["sampled_ids"], b["mu_logp"], b["advantages"], delta=b["delta"], variant=b["variant"],
                                  loss_scale=b["loss_scale"])[0]
    torch.autograd.grad(forward(), (h, wt))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.memory_allocated()
    loss = forward()
    torch.cuda.synchronize()
    held = torch.cuda.memory_allocated() - before
    # beside it: the hidden states' gradient and copy, the per-token outputs, and what the allocator adds to a
    # block (up to 1 MiB to each of three large ones)
    slack = 4 * T * d + 64 * T + (3 << 20)
    most = 4 * V * d + max(V * d // 2, A.HELD_MORE)
    assert held <= (most if B.lmhead_workspace_bytes(T, V) + 2 * T * d <= most else 4 * V * d) + slack
    if room:
        assert B.lmhead_workspace_bytes_best(T, V, d) > B.lmhead_workspace_bytes(T, V) + slack
        assert held <= B.lmhead_workspace_bytes(T, V) + slack
    torch.autograd.grad(loss, (h, wt))
