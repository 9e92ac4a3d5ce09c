"""GPU parity of the exact full-vocabulary variants (trust region on the true TV / KL between the
rollout policy's and the trainer's rows, App. B) against the float64 oracle, through the C ABI."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2602_04879_amd import binding as B
from paper_2602_04879_amd import workloads as W
from tests import parity as P
from tests.test_gpu_parity import DEV, _run_and_compare, _say

pytestmark = pytest.mark.gpu

FULL = [(W.FULL_TV, 0.2), (W.FULL_KL, 0.05)]


@pytest.mark.parametrize("variant,delta", FULL)
@pytest.mark.parametrize("shift", [0.0, 2.0])
def test_c1_shape_all_rows(variant, delta, shift):
    w = W.scaled(W.WORKLOADS["c1_tiny_binary_tv"], variant=variant, delta=delta, mu_full=True,
                 noise_std=1.0 if shift else 0.05)
    b, res, st = _run_and_compare(w, shift=shift)
    assert B.last_path() == "fullvocab"
    if shift:
        assert 0 < st["masked"] < b["T"]
    _run_and_compare(w, shift=shift, backward=False)


@pytest.mark.parametrize("variant,delta", FULL)
@pytest.mark.parametrize("V,ld", [(1, 1), (7, 7), (8, 8), (1000, 1000), (5003, 5003), (5003, 5011), (32768, 32768),
                                  (40004, 40010), (151936, 151936)])
def test_ragged_rows_pitches_and_workgroup_sizes(variant, delta, V, ld):
    # V = 1 .. 151936 covers the three workgroup sizes, rows with head / vector / tail parts, odd
    # pitches (rows that change their 16-byte misalignment from one to the next) and a poisoned pad
    w = W.Workload("ragged_full", 3, 5, V, variant, delta, mu_full=True, logit_std=3.0, noise_std=0.7, zipf_s=1.1,
                   adv="normal", seed=53)
    _run_and_compare(w, ld=ld, shift=1.0 if V > 1 else 0.0)
    _run_and_compare(w, ld=ld, in_place=True)


@pytest.mark.parametrize("variant,delta", FULL)
def test_rows_of_the_two_matrices_misaligned_against_each_other(variant, delta):
    """mu_logits with a pitch of its own and a start 2 bytes off: the vector path cannot apply."""
    w = W.Workload("misfull", 2, 9, 4104, variant, delta, mu_full=True, logit_std=3.0, noise_std=0.7, adv="pm1", seed=59)
    b = W.make_batch(w, DEV)
    T, V = b["T"], b["V"]
    store = torch.full((T * (V + 24) + 8,), 1.0e4, dtype=torch.bfloat16, device=DEV)
    mu2 = store[1:1 + T * (V + 24)].view(T, V + 24)[:, :V]
    mu2.copy_(b["mu_logits"][:, :V])
    b["mu_logits"] = mu2
    rows = np.arange(T)
    ref = P.oracle_rows(b, rows)
    res = B.run_batch(b, diagnostics=True)
    torch.cuda.synchronize()
    assert res["args"].mu_ld == V + 24
    st = P.compare_rows(b, res, rows, ref=ref)
    P.check_loss_scalar(b, res, float(ref["loss_tok"].sum()))
    _say(f"       {st}")


@pytest.mark.parametrize("V", [8192, 98312])
def test_excluded_tokens_and_infinite_kl(V):
    """-inf logits: a token both policies exclude adds nothing; one only mu excludes adds nothing to
    KL(mu || pi); one only pi excludes while mu can sample it makes KL infinite (TV stays finite).
    In the general kernel (V = 8192) and in the register-resident form (V = 98312)."""
    for variant, delta in FULL:
        w = W.Workload("inf_full", 2, 6, V, variant, delta, mu_full=True, logit_std=2.0, noise_std=0.3, adv="pm1", seed=61)
        b = W.make_batch(w, DEV)
        a = b["sampled_ids"].long()
        cols = torch.arange(100, 2000, device=DEV)
        keep = [(int(a[r]) < 100 or int(a[r]) >= 2000) for r in range(b["T"])]    # rows whose sampled token stays
        r_both, r_mu, r_pi = [r for r in range(b["T"]) if keep[r]][:3]
        b["logits"][r_both, cols] = float("-inf"); b["mu_logits"][r_both, cols] = float("-inf")
        b["mu_logits"][r_mu, cols] = float("-inf")
        b["logits"][r_pi, cols] = float("-inf")
        rows = np.arange(b["T"])
        ref = P.oracle_rows(b, rows)
        res = B.run_batch(b, diagnostics=True)
        torch.cuda.synchronize()
        assert B.last_path() == ("fullvocab" if V == 8192 else "fullvocab_resident")
        st = P.compare_rows(b, res, rows, ref=ref)
        D = res["divergence"].cpu().numpy()
        if variant == W.FULL_KL:
            assert np.isinf(ref["divergence"][r_pi]) and np.isinf(D[r_pi]) and D[r_pi] > 0
        assert np.isfinite(np.delete(D, r_pi)).all()
        assert torch.isfinite(res["grad_logits"].float()).all()
        _say(f"       variant={variant} {st}")


@pytest.mark.parametrize("variant,delta", FULL)
def test_identical_rows_give_zero_and_special_rows(variant, delta):
    w = W.Workload("same_full", 4, 20, 16384, variant, delta, mu_full=True, logit_std=3.0, noise_std=0.5, zipf_s=1.1,
                   adv="normal", seed=67)
    b = W.make_batch(w, DEV, shift_sampled=1.5)
    b["mu_logits"][:10] = b["logits"][:10]                   # identical policies
    b["sampled_ids"][::7] = -1
    b["advantages"][3::9] = 0.0
    rows = np.arange(b["T"])
    ref = P.oracle_rows(b, rows)
    res = B.run_batch(b, diagnostics=True)
    torch.cuda.synchronize()
    st = P.compare_rows(b, res, rows, ref=ref)
    D = res["divergence"].cpu().numpy()
    live = (b["sampled_ids"][:10] >= 0).cpu().numpy()
    assert np.all(np.abs(D[:10][live]) <= 1e-6)
    assert st["masked"] > 0
    P.check_loss_scalar(b, res, float(ref["loss_tok"].sum()))
    _say(f"       {st}")


def test_every_approximation_lower_bounds_the_exact_divergence_on_the_gpu():
    """App. B at the headline vocabulary: Binary <= Top-K <= exact, token by token, all computed by
    the library on the same batch."""
    w = W.scaled(W.WORKLOADS["c6_qwen3_full_tv"], n_seq=4, seq_len=64, K=20)
    b = W.make_batch(w, DEV, shift_sampled=1.0)
    mu = torch.log_softmax(b["mu_logits"][:, :b["V"]].float(), -1)
    v, i = torch.topk(mu, 20, dim=-1)
    b["mu_topk_ids"], b["mu_topk_logp"], b["K"] = i.to(torch.int32), v.contiguous(), 20
    for chain in ((W.BINARY_TV, W.TOPK_TV, W.FULL_TV), (W.BINARY_KL, W.TOPK_KL, W.FULL_KL)):
        Ds = []
        for variant in chain:
            bb = dict(b, variant=variant)
            res = B.run_batch(bb, backward=False)
            torch.cuda.synchronize()
            Ds.append(res["divergence"].double().cpu().numpy())
        assert np.all(Ds[0] <= Ds[1] + 2e-6) and np.all(Ds[1] <= Ds[2] + 2e-6)
        assert (Ds[2] - Ds[1]).max() > 1e-4          # and the bound is not vacuous on this batch
        _say(f"       chain {chain}: mean D {[float(d.mean()) for d in Ds]}")


def test_error_codes():
    w = W.scaled(W.WORKLOADS["c1_tiny_binary_tv"], variant=W.FULL_TV, mu_full=True)
    b = W.make_batch(w, DEV)
    out = B.alloc_outputs(b["T"], DEV)
    grad = torch.empty_like(b["logits"])

    def status(**kw):
        a = B.make_args(b["logits"], b["sampled_ids"], b["mu_logp"], b["advantages"], b["delta"], W.FULL_TV, 1.0, out,
                        grad_logits=grad, mu_logits=b["mu_logits"])
        for k, v in kw.items():
            setattr(a, k, v)
        return B.lib().dppo_loss_fwd_bwd(C.byref(a), None)

    assert status() == 0
    assert status(mu_logits=None) == 1
    assert status(mu_ld=b["V"] - 1) == 2
    assert status(mu_logits=b["mu_logits"].data_ptr() + 1) == 3
    assert status(variant=6) == 4
    torch.cuda.synchronize()


@pytest.mark.parametrize("name", ["c6_qwen3_full_tv", "c6_qwen3_full_kl"])
def test_full_size_sampled_rows(name):
    """T = 32768, V = 151936 in the launch configuration bench.py times: a sample of rows against
    the oracle (first, last, masked, zero-advantage, random), the loss against the per-token terms."""
    w = W.WORKLOADS[name]
    _say(f"[case] {name} full size")
    b = W.make_batch(w, DEV, rows_per_step=2048)
    grad = torch.empty_like(b["logits"])
    res = B.run_batch(b, grad=grad, diagnostics=True)
    torch.cuda.synchronize()
    assert B.last_path() == "fullvocab_resident"
    mask = res["mask"].cpu().numpy()
    adv = b["advantages"].cpu().numpy()
    rng = np.random.default_rng(5)
    pick = {0, b["T"] - 1}
    pick.update(np.nonzero(mask == 0)[0][:6].tolist())
    pick.update(np.nonzero(adv == 0)[0][:2].tolist())
    pick.update(rng.integers(0, b["T"], 20).tolist())
    rows = np.array(sorted(pick))
    st = P.compare_rows(b, res, rows)
    P.check_loss_scalar(b, res)
    assert 0 < (mask == 0).sum() < b["T"] // 10
    _say(f"       masked={(mask == 0).sum()} {st}")


@pytest.mark.parametrize("variant,delta", FULL)
@pytest.mark.parametrize("V,ld", [(98312, 98312), (128256, 128264), (131072, 131072), (131080, 131080), (150008, 150016),
                                  (155648, 155648)])
def test_resident_form_against_the_oracle_and_the_general_kernel(variant, delta, V, ld):
    """Backward on long aligned rows: the trainer's row is held in registers (both chunk counts, the
    shortest and the longest row of each, rows that end inside a chunk, a pitch with a poisoned pad),
    with ignored, zero-advantage and identical rows, separate and in place, with and without the
    diagnostics; and the general kernel on the same input gives the same masks and divergences."""
    w = W.Workload("fv_resident", 3, 7, V, variant, delta, mu_full=True, logit_std=3.0, noise_std=0.7, zipf_s=1.1,
                   adv="normal", seed=71)
    b = W.make_batch(w, DEV, shift_sampled=1.0, ld=ld)
    b["mu_logits"][:3, :V] = b["logits"][:3, :V]             # identical policies
    b["sampled_ids"][5] = -1
    b["sampled_ids"][6] = V - 1                              # the sampled token in the row's last vector
    b["advantages"][8] = 0.0
    rows = np.arange(b["T"])
    ref = P.oracle_rows(b, rows)
    _say(f"[case] resident full-vocabulary form V={V} ld={ld} variant={variant}")
    res = B.run_batch(b, diagnostics=True, grad=torch.full_like(b["logits"], 77.0))
    torch.cuda.synchronize()
    assert B.last_path() == "fullvocab_resident"
    st = P.compare_rows(b, res, rows, ref=ref)
    P.check_loss_scalar(b, res, float(ref["loss_tok"].sum()))
    assert st["masked"] > 0
    assert (res["grad_logits"][:, V:] == 77.0).all()         # the pad between rows is the caller's
    gen = B.run_batch(b, diagnostics=True, flags=B.FLAG_FORCE_STREAMING)
    torch.cuda.synchronize()
    assert B.last_path() == "fullvocab"
    assert torch.equal(gen["mask"], res["mask"])
    assert (gen["divergence"] - res["divergence"]).abs().max().item() <= 2e-6
    plain = B.run_batch(b)                                   # no diagnostics: the other instantiation
    torch.cuda.synchronize()
    assert torch.equal(plain["mask"], res["mask"]) and torch.equal(plain["divergence"], res["divergence"])
    assert torch.equal(plain["grad_logits"][:, :V], res["grad_logits"][:, :V])
    fwd = B.run_batch(b, backward=False, diagnostics=True)   # forward only: the TV form keeps the trainer's row resident too
    torch.cuda.synchronize()
    assert B.last_path() == ("fullvocab_resident" if variant == W.FULL_TV else "fullvocab")
    assert torch.equal(fwd["mask"], res["mask"]) and (fwd["divergence"] - res["divergence"]).abs().max().item() <= 2e-6
    assert torch.allclose(fwd["loss"], res["loss"], rtol=1e-5, atol=1e-9)
    assert torch.allclose(fwd["diagnostics"], res["diagnostics"], rtol=1e-5, atol=1e-6, equal_nan=True)
    keep = res["grad_logits"][:, :V].clone()
    inp = B.run_batch(b, in_place=True)
    torch.cuda.synchronize()
    assert torch.equal(inp["grad_logits"][:, :V], keep)
    _say(f"       {st}")


def test_resident_form_more_rows_than_workgroups_and_fallbacks():
    """Several rows per persistent workgroup, sampled rows against the oracle; a rollout matrix that
    starts 2 bytes off, a forward-only call and a short row stay with the general kernel."""
    w = W.Workload("fv_many", 20, 30, 98816, W.FULL_KL, 0.05, mu_full=True, logit_std=3.0, noise_std=0.7, zipf_s=1.1,
                   adv="normal", seed=73)
    b = W.make_batch(w, DEV, shift_sampled=1.0)
    b["sampled_ids"][::11] = -1
    res = B.run_batch(b, diagnostics=True)
    torch.cuda.synchronize()
    assert B.last_path() == "fullvocab_resident"
    rows = np.array(sorted(set([0, 1, 255, 256, 257, 511, 512, b["T"] - 1] + np.random.default_rng(3).integers(0, b["T"], 12).tolist())))
    st = P.compare_rows(b, res, rows)
    P.check_loss_scalar(b, res)
    _say(f"       {st}")
    B.run_batch(b, backward=False)                           # forward-only KL reads each row once anyway
    torch.cuda.synchronize()
    assert B.last_path() == "fullvocab"
    tvb = dict(b, variant=W.FULL_TV, delta=0.2)
    tvf = B.run_batch(tvb, backward=False, diagnostics=True)  # forward-only TV, several rows per workgroup, ignored rows
    torch.cuda.synchronize()
    assert B.last_path() == "fullvocab_resident"
    st = P.compare_rows(tvb, tvf, rows, check_grad=False)
    P.check_loss_scalar(tvb, tvf)
    _say(f"       forward-only TV {st}")
    T, V = b["T"], b["V"]
    store = torch.zeros(T * V + 8, dtype=torch.bfloat16, device=DEV)
    mu2 = store[1:1 + T * V].view(T, V)
    mu2.copy_(b["mu_logits"])
    off = B.run_batch(dict(b, mu_logits=mu2))
    torch.cuda.synchronize()
    assert B.last_path() == "fullvocab"
    assert torch.equal(off["mask"], res["mask"]) and (off["divergence"] - res["divergence"]).abs().max().item() <= 2e-6
    short = W.Workload("fv_short", 2, 5, 65536, W.FULL_TV, 0.2, mu_full=True, logit_std=3.0, noise_std=0.7, adv="pm1", seed=79)
    B.run_batch(W.make_batch(short, DEV))
    torch.cuda.synchronize()
    assert B.last_path() == "fullvocab"


@pytest.mark.parametrize("variant,delta", FULL)
@pytest.mark.parametrize("V", [57344, 65536, 73736, 98304, 100000])
def test_rows_handed_out_at_run_time_match_rows_fixed_by_index(variant, delta, V):
    """The gradient forms of the register-resident kernel hand their rows out at run time when each
    workgroup has several: every per-row output bit for bit what the form with rows fixed by the
    workgroup index writes, the scalar loss repeatable bit for bit, a minimum-size workspace falling
    back to fixed rows; ignored and zero-advantage rows included; a sample against the oracle."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    T = (12 if V == 100000 else 16) * cus + 29
    w = W.Workload("dynfull", 1, T, V, variant, delta, mu_full=True, logit_std=3.0, noise_std=0.7, zipf_s=1.1, adv="normal", seed=127)
    b = W.make_batch(w, DEV, shift_sampled=1.0)
    b["advantages"] = torch.randn(T, device=DEV)
    b["sampled_ids"][::17] = -1
    b["advantages"][5::19] = 0.0
    fixed = B.run_batch(b, diagnostics=True, flags=B.FLAG_STATIC_ROWS)
    assert B.last_path() == "fullvocab_resident"
    runs = [B.run_batch(b, diagnostics=True) for _ in range(3)]
    small = B.alloc_outputs(T, DEV, want_diagnostics=True)
    small["workspace"] = torch.empty(B.WORKSPACE_BYTES, dtype=torch.uint8, device=DEV)
    rmin = B.run_batch(b, out=small)
    torch.cuda.synchronize()
    assert B.last_path() == "fullvocab_resident"
    for r in runs + [rmin]:
        for k in ("loss_tok", "divergence", "mask", "diagnostics", "grad_logits"):
            assert torch.equal(fixed[k], r[k]), k
    for r in runs[1:]:
        assert torch.equal(runs[0]["loss"], r["loss"])
    assert torch.equal(fixed["loss"], rmin["loss"])
    assert abs(runs[0]["loss"].item() - fixed["loss"].item()) <= 1e-6 * abs(fixed["loss"].item())
    plain, plain_fixed = B.run_batch(b), B.run_batch(b, flags=B.FLAG_STATIC_ROWS)        # (without diagnostics)
    torch.cuda.synchronize()
    assert torch.equal(plain["grad_logits"], plain_fixed["grad_logits"]) and torch.equal(plain["divergence"], fixed["divergence"])
    rows = np.arange(T)[::24 if V == 100000 else 96]
    st = P.compare_rows(b, runs[0], rows)
    assert 0 < (runs[0]["mask"] == 0).sum().item() < T
    _say(f"       {st}")


@pytest.mark.parametrize("variant,delta", FULL)
@pytest.mark.parametrize("V", [4096, 151936])
def test_mask_anchored_to_a_recomputed_policy(variant, delta, V):
    """anchor_logp with the exact divergences (both kernels): the direction test of the mask looks at
    the anchor (the divergence is that of the two rows given, whichever policy the second one is)."""
    w = W.Workload("full_anchor", 2, 20, V, variant, delta, mu_full=True, logit_std=3.0, noise_std=1.0, adv="normal", seed=101)
    b = W.make_batch(w, DEV, shift_sampled=2.0)
    g = torch.Generator(device="cpu").manual_seed(9)
    b["anchor_logp"] = torch.minimum(b["mu_logp"] + torch.randn(b["T"], generator=g).to(DEV) * 1.5, torch.zeros_like(b["mu_logp"]))
    rows = np.arange(b["T"])
    ref = P.oracle_rows(b, rows)
    res = B.run_batch(b, diagnostics=True)
    torch.cuda.synchronize()
    assert B.last_path() == ("fullvocab_resident" if V > 100000 else "fullvocab")
    st = P.compare_rows(b, res, rows, ref=ref)
    P.check_loss_scalar(b, res, float(ref["loss_tok"].sum()))
    res0 = B.run_batch(dict(b, anchor_logp=None))
    torch.cuda.synchronize()
    assert (res0["mask"] != res["mask"]).any()
    _say(f"       {st}")


@pytest.mark.parametrize("variant,delta", FULL)
@pytest.mark.parametrize("V,ld", [(8200, 8200), (12296, 12352), (16384, 16384), (20488, 20488), (32000, 32000), (36872, 36872), (49152, 49152),
                                  (49160, 49160), (57344, 57344), (61440, 61440), (65536, 65536), (73736, 73736), (98304, 98304)])
def test_resident_form_on_shorter_rows(variant, delta, V, ld):
    """Every shape of the register-resident form below 98312 entries, at its shortest or longest row:
    several rows per workgroup, ignored, masked and zero-advantage rows, identical policies, sampled tokens at both ends,
    a poisoned pitch that stays untouched; a sample against the oracle, all rows against the general kernel, in
    place, and run after run the same bits."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    # (the KL form with one workgroup per compute unit and a short row: up to four rows each)
    T = 3 * cus + 37 if variant == W.FULL_KL and 49152 < V < 65536 else 4 * cus + 37
    w = W.Workload("fv_mid", 1, T, V, variant, delta, mu_full=True, logit_std=3.0, noise_std=0.7, zipf_s=1.1, adv="normal", seed=137)
    b = W.make_batch(w, DEV, shift_sampled=1.0, ld=ld, rows_per_step=512)
    b["advantages"] = torch.randn(T, device=DEV)
    b["mu_logits"][:3, :V] = b["logits"][:3, :V]
    b["sampled_ids"][7::17] = -1
    b["sampled_ids"][8], b["sampled_ids"][9], b["sampled_ids"][T - 1] = V - 1, 0, V - 8
    b["advantages"][5::19] = 0.0
    b["logits"][10, 100:4000] = float("-inf"); b["mu_logits"][10, 100:4000] = float("-inf")
    b["sampled_ids"][10] = 5
    _say(f"[case] resident full-vocabulary form, shorter rows V={V} ld={ld} variant={variant}")
    res = B.run_batch(b, diagnostics=True, grad=torch.full_like(b["logits"], 77.0))
    torch.cuda.synchronize()
    taken = variant == W.FULL_TV or V not in (8200, 49152, 49160)       # the KL form: where it is the faster one
    assert B.last_path() == ("fullvocab_resident" if taken else "fullvocab")
    assert (res["grad_logits"][:, V:] == 77.0).all()
    rows = np.array(sorted(set(list(range(12)) + [T - 1, T - 2, 2 * cus, 2 * cus + 1] + np.random.default_rng(3).integers(0, T, 8).tolist())))
    st = P.compare_rows(b, res, rows)
    P.check_loss_scalar(b, res)
    gen = B.run_batch(b, diagnostics=True, flags=B.FLAG_FORCE_STREAMING)
    again = B.run_batch(b, diagnostics=True)
    torch.cuda.synchronize()
    assert torch.equal(gen["mask"], res["mask"])
    assert (gen["divergence"] - res["divergence"]).abs().max().item() <= 2e-6
    for k in ("loss", "loss_tok", "divergence", "mask", "diagnostics"):
        assert torch.equal(again[k], res[k]), k
    assert torch.equal(again["grad_logits"][:, :V], res["grad_logits"][:, :V])
    keep = res["grad_logits"][:, :V].clone()
    plain = B.run_batch(b, in_place=True)
    torch.cuda.synchronize()
    assert torch.equal(plain["grad_logits"][:, :V], keep) and torch.equal(plain["divergence"], res["divergence"])
    assert 0 < (res["mask"] == 0).sum().item() < T
    _say(f"       {st}")


@pytest.mark.parametrize("variant,delta", FULL)
@pytest.mark.parametrize("V", [12296, 16384, 24576, 32000])
def test_short_rows_whose_largest_entry_is_anywhere(variant, delta, V):
    """Rows short enough that a thread knows its largest entry before its first exponential: the largest entry of a row in
    every position of a 16-byte block and far above the rest, rows of one sign, blocks of -inf, and -0.  (Both rows
    alike in size: the cross term of the KL form, a sum in fp32, loses what the rows differ by.)"""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    T = cus + 40
    w = W.Workload("fv_max", 1, T, V, variant, delta, mu_full=True, logit_std=3.0, noise_std=0.7, adv="normal", seed=139)
    b = W.make_batch(w, DEV, shift_sampled=1.0, rows_per_step=512)
    b["advantages"] = torch.randn(T, device=DEV)
    z, y = b["logits"], b["mu_logits"]
    for t in range(16):                               # 8 positions in a block, in the first and the last chunk
        j = (t if t < 8 else V - 16 + t) if t % 2 else (4096 + t if t < 8 else V - 24 + t)
        z[t, j], y[t, j] = 20.0 + t, 20.5 + t
        if t % 3 == 0:
            b["sampled_ids"][t] = j
    z[16], y[16] = -1.0 - z[16].abs(), -1.0 - y[16].abs()
    z[17], y[17] = z[17] - 30.0, y[17] - 30.0
    z[18, 64:V - 64] = float("-inf"); y[18, 64:V - 64] = float("-inf")
    z[19], y[19] = -0.0, 0.0
    z[20], y[20] = -0.0, -1.0
    z[18, :8], y[18, :8] = -5.0, -6.0
    b["sampled_ids"][18], b["sampled_ids"][16:18] = 3, 7
    rows = np.arange(24)
    _say(f"[case] exact divergence, largest entries anywhere V={V} variant={variant}")
    res = B.run_batch(b, diagnostics=True)
    torch.cuda.synchronize()
    if variant == W.FULL_TV or V != 12296:              # (the KL form: rows that fill their shape)
        assert B.last_path() == "fullvocab_resident"
    gen = B.run_batch(b, diagnostics=True, flags=B.FLAG_FORCE_STREAMING)
    torch.cuda.synchronize()
    st = P.compare_rows(b, res, rows)
    ok = torch.isfinite(gen["divergence"])
    assert torch.equal(ok, torch.isfinite(res["divergence"]))
    # both sides within the module's bound of the oracle: 1e-4 relative + 3e-7, each
    assert ((gen["divergence"] - res["divergence"]).abs()[ok] <= 2e-4 * gen["divergence"][ok] + 6e-7).all()
    _say(f"       {st}")


@pytest.mark.parametrize("variant,delta", FULL)
def test_every_row_whatever_number_is_left_over(variant, delta):
    """Two workgroups per compute unit, rows fixed by the workgroup index: one round exactly and less, one
    row left over, all but one, several rounds.  Every row is written, with the bits that it has in a call of
    other size."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    T = 6 * cus + 1
    w = W.Workload("fv_left", 1, T, 16384, variant, delta, mu_full=True, logit_std=3.0, noise_std=0.7, adv="normal", seed=139)
    b = W.make_batch(w, DEV, shift_sampled=1.0, rows_per_step=1024)
    b["sampled_ids"][3::29] = -1
    per_row = ("logits", "mu_logits", "sampled_ids", "mu_logp", "advantages")
    want = None
    for n in (T, cus, 2 * cus - 1, 2 * cus, 2 * cus + 1, 2 * cus + 88, 4 * cus - 1, 4 * cus, 6 * cus - 1):
        _say(f"[case] rows left over T={n} variant={variant}")
        part = dict(b, T=n, **{k: b[k][:n] for k in per_row})
        out = B.alloc_outputs(n, DEV)
        for k in ("loss_tok", "divergence"):
            out[k].fill_(77.0)
        out["mask"].fill_(77)
        res = B.run_batch(part, out=out, grad=torch.full_like(part["logits"], 77.0))
        torch.cuda.synchronize()
        assert B.last_path() == "fullvocab_resident"
        P.check_loss_scalar(part, res)
        if want is None:
            want = {k: res[k].clone() for k in ("loss_tok", "divergence", "mask", "grad_logits")}
            P.compare_rows(part, res, np.array([0, 1, 3, 2 * cus, 4 * cus, T - 1]))
            assert not (want["grad_logits"][3] != 0).any()
        for k, v in want.items():
            assert torch.equal(res[k], v[:n]), k
