"""The masked layout (one class in position order, memberships tested per pair), which short sequences take, at the
sizes where its tiles and words end; and the class-tile kernels, which the size estimate keeps for longer sequences,
on the small shapes where every row can be checked."""
import numpy as np
import pytest
import torch

from oracle import focus_oracle as fo
from paper_2604_03260_amd import focus, workloads
from tests import harness
from tests import test_gpu_instantiations as inst

pytestmark = pytest.mark.gpu


def _check(wl, inp=None):
    inp = inp if inp is not None else workloads.make_inputs(wl, "cuda")
    res = harness.run_gpu(wl, inp)
    mq, mk = harness.check_assign(wl, inp, res)
    harness.check_attn(wl, inp, res, mq, mk)
    harness.check_pair_totals(wl, res, mq, mk)
    return res


# n around the 32-key units, 64-key tiles, 128-row tiles and 256-position sort blocks; windows of one key, inside a
# unit, across units and tiles, nearly everything; one, two and more groups per token (the word loop past two groups)
@pytest.mark.parametrize("n", [2, 31, 33, 64, 65, 127, 129, 257, 300])
@pytest.mark.parametrize("w,K,topk,causal,dtype,d,softcap", [
    (1, 4, 1, True, "bf16", 64, 0.0), (29, 8, 2, True, "bf16", 128, 0.0), (70, 8, 4, False, "f16", 80, 0.0),
    (1, 16, 2, False, "bf16", 64, 0.0), (250, 32, 5, True, "bf16", 96, 30.0), (64, 32, 2, True, "bf16", 256, 0.0),
    (33, 8, 1, True, "f32", 64, 0.0)])
def test_masked_tile_edges(n, w, K, topk, causal, dtype, d, softcap):
    if w >= n:
        w = max(1, n - 1)
    _check(workloads.Workload("m", 300 + n, 1, 4, 2, n, d, dtype, K, topk, w, causal=causal, softcap=softcap, mixture=3))


# the same edges with enough heads that the tiles run instead of the kernel for a few work-groups of 32 rows
@pytest.mark.parametrize("n", [2, 33, 65, 129, 257])
@pytest.mark.parametrize("w,K,topk,causal,dtype,d,softcap", [
    (1, 4, 1, True, "bf16", 64, 0.0), (29, 8, 2, True, "bf16", 128, 0.0), (70, 8, 4, False, "f16", 80, 0.0),
    (1, 16, 2, False, "bf16", 64, 0.0), (250, 32, 5, True, "bf16", 96, 30.0)])
def test_masked_tile_edges_many_heads(n, w, K, topk, causal, dtype, d, softcap):
    if w >= n:
        w = max(1, n - 1)
    wl = workloads.Workload("m", 310 + n, 8, 64, 8, n, d, dtype, K, topk, w, causal=causal, softcap=softcap, mixture=3)
    inp = workloads.make_inputs(wl, "cuda")
    res = harness.run_gpu(wl, inp)
    mq, mk = harness.check_assign(wl, inp, res)
    harness.check_pair_totals(wl, res, mq, mk)
    o_ref, l_ref, pairs = fo.attn_rows(harness.problem_of(wl), *harness.host_inputs(inp), mq, mk)
    flat = lambda t: t.reshape((-1,) + tuple(t.shape[3:])).double().cpu().numpy()
    assert np.array_equal(flat(res["row_pairs"]).astype(np.int64), pairs)
    # Rounding the scaled query row (one half ulp, 2^-9 or 2^-12, per component) moves a logit by at most that times
    # scale * |q| * |k|, and with the rounding of the probabilities (one half ulp more) lse by no more than the logit that
    # moves most.  In rows of one or two keys nothing averages: an output moves by at most max|v| times that, plus its own
    # rounding.  q: the row's own, k and v: the largest that the row may attend.
    half_ulp = {"bf16": 2.0 ** -9, "f16": 2.0 ** -12}[dtype]
    upto = lambda t: t.cummax(dim=2).values if causal else t.amax(dim=2, keepdim=True).expand_as(t)
    per_row = lambda t: upto(t).repeat_interleave(wl.Hq // wl.Hkv, dim=1)
    kmax, vmax = per_row(inp["k"].float().norm(dim=-1)), per_row(inp["v"].float().abs().amax(dim=-1))
    delta = half_ulp * (1.0 + inp["q"].float().norm(dim=-1) * kmax / d ** 0.5)
    few = pairs <= 2
    tol = harness.TOL[dtype]
    lse_tol = np.maximum(tol["lse"], flat(delta))
    out_tol = np.where(few, np.maximum(tol["out_max"], flat(vmax * (delta + half_ulp))), tol["out_max"])
    err = np.abs(flat(res["out"]) - o_ref)
    assert (err.max(axis=-1) <= out_tol).all() and err.mean() <= tol["out_mean"]
    assert (np.abs(flat(res["lse"]) - l_ref) <= lse_tol).all()


CASES_M = [c for c in inst.CASES4 if not c[4]]


@pytest.mark.parametrize("d,softcap,pairs,dtype,coarse,noref", CASES_M)
def test_masked_instantiations_all_rows(d, softcap, pairs, dtype, coarse, noref):
    """Every compiled form of the tiled kernel on the masked layout (24 heads: more than the short kernel takes)."""
    wl = workloads.Workload("instm", 94, 3, 8, 2, 520 + d // 4, d, dtype, 8, 3, 48, softcap=50.0 if softcap else 0.0, mixture=4)
    inst.run_case(wl, pairs, big_norms=not noref)


@pytest.mark.parametrize("B", [1, 20])
def test_masked_rows_with_large_norms_take_the_running_reference(B):
    """Key norms past the bound of the form without a reference: disallowed keys with the largest logits must not
    move the row's reference (their probabilities would drown the allowed ones)."""
    wl = workloads.Workload("m", 331, B, 2, 1, 400, 64, "bf16", 4, 1, 16)
    inp = workloads.make_inputs(wl, "cuda")
    inp["q"] *= 8.0
    inp["k"] *= 8.0
    p = harness.params_of(wl)
    ws = focus.alloc_workspace(p)
    outs = []
    for vector in (False, True):
        out, lse = torch.empty_like(inp["q"]), torch.empty((B, 2, 400), dtype=torch.float32, device="cuda")
        focus.focus_assign(p, inp["q"], inp["k"], inp["centroids"], ws)
        focus.focus_attn_fwd(p, inp["q"], inp["k"], inp["v"], ws, out, lse, vector=vector)
        outs.append((out.float(), lse))
    # logits reach a few hundred: one bf16 ulp of the output (2^-8 relative, values up to 4) and fp32 logits
    assert (outs[0][0] - outs[1][0]).abs().max() <= 2e-2
    assert ((outs[0][1] - outs[1][1]).abs() / outs[1][1].abs().clamp(min=1.0)).max() <= 1e-4


@pytest.mark.parametrize("d,softcap,pairs,dtype,coarse,noref", inst.CASES4)
def test_class_tiles_all_rows(d, softcap, pairs, dtype, coarse, noref, monkeypatch):
    """The same shapes as one pass over class-ordered tiles (exact and coarse classes)."""
    monkeypatch.setenv("FOCUS_TWO_PASS", "0")
    inst.test_four_wavefront_instantiations_all_rows(d, softcap, pairs, dtype, coarse, noref)


@pytest.mark.parametrize("n,K,topk,w", [(777, 4, 2, 32), (1500, 32, 2, 40), (700, 16, 3, 16), (2000, 12, 3, 30)])
def test_class_tiles_against_the_masked_layout(n, K, topk, w, monkeypatch):
    """Both layouts of one problem: equal memberships, pair counts and (to rounding) outputs."""
    wl = workloads.Workload("m", 340, 1, 4, 2, n, 128, "bf16", K, topk, w, mixture=4)
    inp = workloads.make_inputs(wl, "cuda")
    masked = _check(wl, inp)
    monkeypatch.setenv("FOCUS_TWO_PASS", "0")
    classes = _check(wl, inp)
    assert torch.equal(masked["row_pairs"], classes["row_pairs"])


@pytest.mark.parametrize("dtype,d,B", [("bf16", 128, 1), ("bf16", 128, 6), ("f16", 80, 1), ("f16", 80, 6), ("bf16", 64, 1), ("f32", 64, 1), ("f32", 256, 1)])
def test_spoiled_values_reach_only_the_rows_that_attend_them(dtype, d, B):
    """V rows with NaN or infinities: the masked tiles visit every key of the causal prefix, with probability zero
    where the pair is not allowed, and 0 * inf must not spoil those rows."""
    wl = workloads.Workload("m", 350, B, 4, 2, 700, d, dtype, 8, 1, 40, mixture=3)
    inp = workloads.make_inputs(wl, "cuda")
    bad_keys = (3, 100, 333, 500)
    for j, x in zip(bad_keys, (float("nan"), float("inf"), -float("inf"), float("inf"))):
        inp["v"][0, 0, j, (7 * j) % d] = x
    res = harness.run_gpu(wl, inp)
    mq, mk = harness.check_assign(wl, inp, res)
    rows, attending = [], []
    for h in range(wl.Hq):
        for i in range(wl.n):
            hit = h < 2 and any(j <= i and (i - j < wl.window or (int(mq[0, h, i]) & int(mk[0, 0, j]))) for j in bad_keys)
            (attending if hit else rows).append((0, h, i))
    assert len(rows) > 1000 and len(attending) > 100
    inp["v"] = torch.nan_to_num(inp["v"], nan=0.0, posinf=0.0, neginf=0.0)         # (for the oracle)
    harness.check_attn(wl, inp, res, mq, mk, rows=np.array(rows, dtype=np.int32))
    at = torch.tensor(attending, device="cuda")
    assert not torch.isfinite(res["out"][at[:, 0], at[:, 1], at[:, 2]].float()).all(dim=-1).any()


# the fp32 kernel at the edges of its 32-row quarters, 32-key units and the round-robin of its four wavefronts, in
# class tiles and in the masked layout (test_masked_tile_edges), every head dim
@pytest.mark.parametrize("n", [1, 32, 33, 95, 129, 400])
@pytest.mark.parametrize("d,K,topk,w,causal,softcap,tiles", [
    (64, 4, 2, 17, True, 0.0, "0"), (80, 8, 3, 40, True, 0.0, None), (96, 16, 3, 25, False, 5.0, "0"),
    (128, 4, 1, 64, True, 0.0, "0"), (256, 8, 2, 33, False, 0.0, None), (128, 2, 2, 500, True, 0.0, None)])
def test_f32_kernel_edges(n, d, K, topk, w, causal, softcap, tiles, monkeypatch):
    if tiles:
        monkeypatch.setenv("FOCUS_TWO_PASS", tiles)
    _check(workloads.Workload("m", 360 + n, 2, 4, 2, n, d, "f32", K, topk, w, causal=causal, softcap=softcap, mixture=2))
