"""The calls this library is timed on: what a trainer has it do, through its public entry points.

Two families.  `logits`: the loss (and its gradient) of one micro-batch whose [T, V] bf16 logits the
trainer holds, through the C ABI's binding with the argument struct kept (`entry` "abi"), or through
the autograd wrapper (`entry` "autograd", the gradient scaled by `upstream`, 1 unless the trainer
weights the loss).  `hidden`: the same from the final hidden states and the lm_head weight, through
the autograd wrapper, both gradients or none.  Sizes are those of the repository's own workloads,
tests and vocabulary sweep; inputs are drawn by its own seeded generators.
"""
import math

import torch

from paper_2602_04879_amd import autograd as A
from paper_2602_04879_amd import binding as B
from paper_2602_04879_amd import workloads as W

DEV = "cuda:0"

# Every field a case can have, with what it is where a case does not say.
DEFAULTS = {
    "family": "logits", "entry": "abi", "backward": True, "T": 256, "V": 4096, "pitch": 0, "d": 0, "variant": W.BINARY_TV, "K": 0,
    "delta": 0.2, "diagnostics": False, "mask_rule": B.MASK_DIVERGENCE, "upstream": 1.0, "zipf": 1.1, "noise": 0.05,
}
TOPK = (W.TOPK_TV, W.TOPK_KL)
FULL = (W.FULL_TV, W.FULL_KL)


def listed():
    return [
        # The smallest configuration of the repository, 4 responses of 64 tokens: latency and launches.
        {"name": "tiny_call", "T": 256, "V": 4096, "zipf": 0.0},
        # What is left of a batch after the full micro-batches: few tokens over a large vocabulary.
        {"name": "short_remainder", "T": 100, "V": 151936, "variant": W.TOPK_TV, "K": 20},
        # 16 responses of 512 tokens over a vocabulary of middle size, KL trust region.
        {"name": "mid_vocab_kl", "T": 8192, "V": 32768, "variant": W.BINARY_KL, "delta": 0.1, "zipf": 0.0, "noise": 0.1},
        # The full-size training step, 16 x 2048 tokens, with the rollout engine's top 20.
        {"name": "step_topk_tv", "T": 32768, "V": 151936, "variant": W.TOPK_TV, "K": 20},
        # The same loss inside a trainer: autograd, odd vocabulary, the baseline's clip mask, and the
        # loss weighted by one over the number of accumulated micro-batches.
        {"name": "autograd_odd_vocab", "entry": "autograd", "T": 6000, "V": 50257, "mask_rule": B.MASK_RATIO_CLIP, "upstream": 0.25},
        # Monitoring pass: no gradient, per-token health metrics, the longest top-K of the workloads.
        {"name": "monitor_forward", "backward": False, "T": 8192, "V": 151936, "variant": W.TOPK_KL, "K": 64, "delta": 0.05,
         "diagnostics": True, "noise": 0.1},
        # The largest vocabulary of the workloads, one micro-batch, through autograd.
        {"name": "vocab_256k", "entry": "autograd", "T": 4096, "V": 256000},
        # Trust region on the exact divergence, both rows at hand: large and middle vocabulary.
        {"name": "exact_kl", "T": 4096, "V": 151936, "variant": W.FULL_KL, "delta": 0.05},
        {"name": "exact_tv_mid_vocab", "T": 8192, "V": 32000, "variant": W.FULL_TV},
        # From the hidden states: a large micro-batch, a small one of a smaller model, and old-policy
        # log-probs without a gradient.
        {"name": "hidden_train", "family": "hidden", "entry": "autograd", "T": 8192, "V": 151936, "d": 4096, "zipf": 0.0},
        {"name": "hidden_train_small", "family": "hidden", "entry": "autograd", "T": 1000, "V": 151936, "d": 2048, "zipf": 0.0,
         "variant": W.TOPK_TV, "K": 20},
        {"name": "hidden_forward", "family": "hidden", "entry": "autograd", "backward": False, "T": 2048, "V": 151936, "d": 2048, "zipf": 0.0},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    c = {"variant": rng.choice([W.BINARY_TV, W.BINARY_TV, W.BINARY_KL, W.TOPK_TV, W.TOPK_KL])}
    if rng.random() < 0.3:
        c.update(family="hidden", entry="autograd", zipf=0.0, backward=rng.random() < 0.75)
        c["V"] = rng.choice([32768, 151936, 64 * _log_uniform(rng, 250, 2400)])
        c["d"] = 64 * _log_uniform(rng, 12, 64)
        c["T"] = _log_uniform(rng, 64, 8192)
    else:
        c["backward"] = rng.random() < 0.85
        c["entry"] = rng.choice(["abi", "abi", "autograd"])
        # the repository's vocabularies, or any other: multiples of 64 (padded embeddings) and odd ones
        v = _log_uniform(rng, 4096, 262144)
        c["V"] = rng.choice([4096, 32768, 50257, 151643, 151936, 256000, min(64 * (v // 64), 262144), v | 1])
        if c["V"] % 64 and rng.random() < 0.3:
            c["pitch"] = 64 * (c["V"] // 64 + 1)         # the padding sliced off: rows on lines, an odd length
        # tokens: from a remainder of a few dozen to the largest listed call
        most = min(131072, 32768 * 151936 // c["V"])
        c["T"] = _log_uniform(rng, 48, most)
        if rng.random() < 0.2 and c["T"] * c["V"] * 1.5 < 32768 * 151936:
            c["variant"] = rng.choice(list(FULL))
        c["diagnostics"] = rng.random() < 0.2
        c["mask_rule"] = rng.choice([B.MASK_DIVERGENCE, B.MASK_DIVERGENCE, B.MASK_RATIO_CLIP])
        if c["entry"] == "autograd" and c["backward"]:
            c["upstream"] = rng.choice([1.0, 1.0, 0.25])
    if c["variant"] in TOPK:
        c["K"] = rng.choice([20, 20, 64, rng.randint(1, 100)])
    if c["variant"] in (W.BINARY_KL, W.TOPK_KL, W.FULL_KL):
        c["delta"] = 0.05
    return c


def _full(case):
    return {**DEFAULTS, **case}


def prepare(case, seed):
    c = _full(case)
    T = c["T"]
    # one response per 64 tokens or so: advantages are per response
    n_seq = next(n for n in range(max(2, T // 64), 0, -1) if T % n == 0)
    w = W.Workload("case", n_seq, T // n_seq, c["V"], c["variant"], c["delta"], K=c["K"], logit_std=3.0, noise_std=c["noise"],
                   zipf_s=c["zipf"], drift_frac=0.05, drift_std=1.5, mu_full=c["variant"] in FULL, d_model=c["d"], adv="normal", seed=seed)
    rows = max(1, min(1024, (1 << 27) // c["V"]))
    if c["family"] == "hidden":
        b = W.make_lmhead_batch(w, c["d"], DEV, rows_per_step=rows)
        if c["backward"]:
            b["hidden"].requires_grad_(True)
            b["weight"].requires_grad_(True)
        return {"case": c, "batch": b}
    b = W.make_batch(w, DEV, ld=c["pitch"] or None, rows_per_step=rows)
    s = {"case": c, "batch": b, "logits": b["logits"][:, : c["V"]]}
    if c["entry"] == "abi":
        s["out"] = B.alloc_outputs(T, DEV, want_diagnostics=c["diagnostics"])
        if c["backward"]:
            s["grad"] = torch.empty_like(b["logits"])[:, : c["V"]]
        s["args"] = B.make_args(s["logits"], b["sampled_ids"], b["mu_logp"], b["advantages"], c["delta"], c["variant"], b["loss_scale"],
                                s["out"], b["mu_topk_ids"], b["mu_topk_logp"], grad_logits=s.get("grad"), mask_rule=c["mask_rule"],
                                eps_low=0.2, eps_high=0.28, mu_logits=b["mu_logits"])
    elif c["backward"]:
        s["logits"] = s["logits"].detach().requires_grad_(True)
    return s


def _picked(out, c):
    return {k: out[k] for k in ("loss", "loss_tok", "divergence", "mask") + (("diagnostics",) if c["diagnostics"] else ())}


def run(state):
    c, b = state["case"], state["batch"]
    if c["entry"] == "abi":
        (B.dppo_loss_fwd_bwd if c["backward"] else B.dppo_loss_fwd)(state["args"])
        out = _picked(state["out"], c)
        if c["backward"]:
            out["grad_logits"] = state["grad"]
        return out
    tk = dict(mu_topk_ids=b["mu_topk_ids"], mu_topk_logp=b["mu_topk_logp"])
    kw = dict(delta=c["delta"], variant=c["variant"], loss_scale=b["loss_scale"], mask_rule=c["mask_rule"], eps_low=0.2, eps_high=0.28,
              diagnostics=c["diagnostics"], **tk)
    side = (b["sampled_ids"], b["mu_logp"], b["advantages"])
    with torch.set_grad_enabled(c["backward"]):
        if c["family"] == "hidden":
            inputs = {"grad_hidden": b["hidden"], "grad_weight": b["weight"]}
            loss, aux = A.dppo_lmhead_loss(b["hidden"], b["weight"], *side, **kw)
        else:
            inputs = {"grad_logits": state["logits"]}
            loss, aux = A.dppo_loss(state["logits"], *side, mu_logits=b["mu_logits"], **kw)
    out = _picked(dict(aux, loss=loss.detach()), c)
    if c["backward"]:
        total = loss if c["upstream"] == 1.0 else loss * c["upstream"]
        out.update(zip(inputs, torch.autograd.grad(total, list(inputs.values()))))
    return out


def work(case):
    c = _full(case)
    T, V, K, d = c["T"], c["V"], c["K"], c["d"]
    # per token: sampled id, log mu, advantage, loss term, divergence (4 bytes each), mask, top-K ids and log-probs
    side = T * (21 + 8 * K + (32 if c["diagnostics"] else 0))
    if c["family"] == "hidden":
        # hidden states and weight in, their gradients out (all bf16); one product, with the gradients three
        n = 2 if c["backward"] else 1
        return {"bytes": side + n * 2 * (T * d + V * d), "flops": (3 if c["backward"] else 1) * 2 * T * V * d}
    rows = 1 + (1 if c["backward"] else 0) + (1 if c["variant"] in FULL else 0)
    # per entry: one multiply-add and one exponential for the softmax, the same for the gradient and the second row
    return {"bytes": side + rows * 2 * T * V, "flops": rows * 3 * T * V}


def tolerance(case):
    c = _full(case)
    if c["family"] == "hidden":
        # logits are rounded to bf16 once: another order of the contraction's fp32 sum rounds a few of
        # them to the neighbour, and a token whose divergence then crosses delta changes its mask
        return {"rel": 0.01 if c["backward"] else 0.005, "max": 0.05, "differ": 0.003}
    if c["backward"]:
        return {"rel": 0.007, "max": 0.016, "differ": 0.0}         # the gradient is rounded to bf16 (and again when scaled)
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}


# ---- the same quantities in 64 bits, from the definitions -------------------------------------------


def _xlogx(x, lx, ly):
    """x (ln x - ln y) with 0 ln 0 = 0, the logarithm of a vanishing y floored."""
    return torch.where(x > 0, x * (lx - ly.clamp(min=math.log(1e-30))), torch.zeros_like(x))


def _rows(c, z, y, a, lmu, adv, tki, tkl, scale):
    """Per-token outputs of rows of float64 logits z [n, V]; also the gradient's two factors (coefficient, softmax)."""
    a = a.long()[:, None]
    lp = torch.log_softmax(z, -1)
    p = lp.exp()
    la, lmu, adv = lp.gather(1, a).squeeze(1), lmu.double(), adv.double()
    qa, pa = la.exp(), lmu.clamp(max=0).exp()
    r = (la - lmu).exp()
    mass_mu, mass_pi = pa, qa
    v = c["variant"]
    if v in FULL:
        lm = torch.log_softmax(y, -1)
        m = lm.exp()
        div = 0.5 * (m - p).abs().sum(-1) if v == W.FULL_TV else (m * (lm - lp)).sum(-1)
        mass_mu = mass_pi = torch.ones_like(pa)
    elif v == W.BINARY_TV:
        div = (pa - qa).abs()
    elif v == W.BINARY_KL:
        op = -torch.expm1(lmu.clamp(max=0))
        oq = p.scatter(1, a, 0.0).sum(-1)
        div = _xlogx(pa, lmu.clamp(max=0), la) + _xlogx(op, op.clamp(min=1e-300).log(), oq.clamp(min=1e-300).log())
    else:
        other = tki.long() != a
        lk, lq = tkl.double().clamp(max=0), lp.gather(1, tki.long())
        pk, qk = torch.where(other, lk.exp(), 0.0), torch.where(other, lq.exp(), 0.0)
        mass_mu, mass_pi = pa + pk.sum(-1), qa + qk.sum(-1)
        po, qo = (1 - mass_mu).clamp(min=0), (1 - mass_pi).clamp(min=0)
        if v == W.TOPK_TV:
            div = 0.5 * ((pa - qa).abs() + (pk - qk).abs().sum(-1) + (po - qo).abs())
        else:
            div = (_xlogx(pa, lmu.clamp(max=0), la) + _xlogx(pk, lk, lq).sum(-1)
                   + _xlogx(po, po.clamp(min=1e-300).log(), qo.clamp(min=1e-300).log()))
    up, down = adv > 0, adv < 0
    if c["mask_rule"] == B.MASK_RATIO_CLIP:
        blocked = (up & (la - lmu > math.log1p(0.28))) | (down & (la - lmu < math.log1p(-0.2)))
    else:
        blocked = (div > c["delta"]) & ((up & (la > lmu)) | (down & (la < lmu)))
    w = torch.where(blocked, 0.0, r * adv)
    out = {"divergence": div, "loss_tok": -w, "mask": (~blocked).to(torch.uint8)}
    if c["diagnostics"]:
        ent = -(p * lp).sum(-1)
        zero = torch.zeros_like(qa)
        out["diagnostics"] = torch.stack([r, la, (pa - qa).abs(), ent, mass_mu, mass_pi, zero, zero], 1)
    return out, scale * w, p, a


@torch.no_grad()
def exact(case, seed):
    s = prepare(case, seed)
    c, b = s["case"], s["batch"]
    T, V = c["T"], c["V"]
    hidden = c["family"] == "hidden"
    up = c["upstream"]
    h = wt = gh = gw = g = None
    if hidden:
        h, wt = b["hidden"].double(), b["weight"].double()
        if c["backward"]:
            gh, gw = torch.empty_like(h), torch.zeros_like(wt)
    elif c["backward"]:
        g = torch.empty((T, V), dtype=torch.float64, device=DEV)
    parts = []
    step = max(1, min(2048, (1 << 28) // V))
    for r0 in range(0, T, step):
        sl = slice(r0, min(T, r0 + step))
        # from the hidden states the logits are DEFINED as the product rounded once to bf16
        z = (h[sl] @ wt.T).to(torch.bfloat16).double() if hidden else b["logits"][sl, :V].double()
        y = b["mu_logits"][sl, :V].double() if c["variant"] in FULL else None
        tki, tkl = (b["mu_topk_ids"][sl], b["mu_topk_logp"][sl]) if c["K"] else (None, None)
        out, coef, p, a = _rows(c, z, y, b["sampled_ids"][sl], b["mu_logp"][sl], b["advantages"][sl], tki, tkl, b["loss_scale"])
        parts.append(out)
        if c["backward"]:
            p.scatter_add_(1, a, torch.full_like(a, -1, dtype=torch.float64))
            p *= (coef * up)[:, None]
            if hidden:
                gh[sl] = p @ wt
                gw += p.T @ h[sl]
            else:
                g[sl] = p
    res = {k: torch.cat([q[k] for q in parts]) for k in parts[0]}
    res["loss"] = (b["loss_scale"] * res["loss_tok"].sum()).reshape(() if c["entry"] == "autograd" else (1,))
    if g is not None:
        res["grad_logits"] = g
    if gh is not None:
        res["grad_hidden"], res["grad_weight"] = gh, gw
    return res
