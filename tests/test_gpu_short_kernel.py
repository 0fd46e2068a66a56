"""The kernel for short 16-bit problems and the fp32 kernel for rows in position order at the edges of its 32-row groups, 32-key units and wavefronts, every head dim; and the
tiled kernel on the masked layout with more heads than the short one takes."""
import pytest
import torch

from paper_2604_03260_amd import focus, workloads
from tests import harness
from tests import test_gpu_f16_range as f16_range
from tests import test_gpu_instantiations as inst
from tests import test_gpu_masked as masked
from tests import test_gpu_nonfinite_values as nonfinite

pytestmark = pytest.mark.gpu


# one unit and less, a wavefront's second unit (from 128 or 256 keys on), a last unit of one key; windows inside a unit and over several
@pytest.mark.parametrize("n", [1, 31, 32, 33, 65, 130, 257, 290])
@pytest.mark.parametrize("d,dtype,K,topk,w,causal,softcap", [
    (64, "f16", 4, 2, 40, True, 5.0), (80, "bf16", 16, 3, 100, True, 0.0), (96, "f16", 8, 1, 7, False, 20.0),
    (128, "bf16", 32, 2, 33, False, 0.0), (256, "bf16", 4, 2, 50, True, 0.0), (256, "f16", 16, 3, 90, False, 30.0), (256, "bf16", 8, 1, 1, True, 0.0),
    (256, "f16", 4, 2, 5000, True, 0.0), (128, "f16", 4, 2, 5000, False, 50.0), (64, "f32", 4, 2, 40, False, 0.0), (80, "f32", 16, 3, 7, True, 20.0),
    (96, "f32", 8, 2, 60, True, 0.0), (128, "f32", 4, 1, 100, True, 0.0), (256, "f32", 32, 2, 33, True, 0.0)])
def test_units_and_groups(n, d, dtype, K, topk, w, causal, softcap):
    masked._check(workloads.Workload("sk", 500 + n, 2, 4, 2, n, d, dtype, K, topk, w, causal=causal, softcap=softcap, mixture=3))


# rows in position order that the fp32 kernel for class tiles walks (by_tiles), at the edges of units
@pytest.mark.parametrize("B,Hq,n,d,w,causal,softcap", [
    (1, 4, 513, 256, 5000, True, 0.0), (1, 3, 545, 256, 5000, False, 20.0), (1, 4, 770, 256, 100, True, 0.0), (1, 12, 650, 256, 90, False, 0.0), (1, 2, 1057, 256, 33, True, 30.0),
    (2, 8, 1030, 96, 60, True, 0.0), (1, 4, 1030, 96, 5000, False, 0.0), (11, 2, 1030, 64, 5000, False, 10.0)])
def test_rows_in_position_order_by_tiles(B, Hq, n, d, w, causal, softcap):
    masked._check(workloads.Workload("sk", 505, B, Hq, Hq // 2 if Hq % 2 == 0 else 1, n, d, "f32", 8, 2, w, causal=causal, softcap=softcap, mixture=3))


@pytest.mark.parametrize("d,dtype,head_map", [(64, "bf16", [1, 0, 0, 1, 2, 2]), (256, "f16", [2, 1, 0, 0, 1, 2]), (80, "f32", [2, 1, 0, 0, 1, 2])])
def test_other_head_maps(d, dtype, head_map):
    wl = workloads.Workload("sk", 501, 2, 6, 3, 200, d, dtype, 8, 2, 30)
    inp = workloads.make_inputs(wl, "cuda")
    res = harness.run_gpu(wl, inp, head_map=head_map)
    mq, mk = harness.oracle_membership(wl, inp, head_map)
    harness.check_attn(wl, inp, res, mq, mk, head_map=head_map)


@pytest.mark.parametrize("n,w,kw", [(700, 300, {}), (642, 5000, dict(K=4, topk=2)), (130, 20, dict(causal=False)), (700, 40, dict(K=16, topk=3)),
                                    (700, 300, dict(pair_set=focus.FOCUS_PAIRS_SHARED)), (700, 60, dict(pair_set=focus.FOCUS_PAIRS_CROSS_LOCAL))])
@pytest.mark.parametrize("dtype,d", [("bf16", 256), ("f16", 96)])
def test_values_that_are_not_finite(dtype, d, n, w, kw):
    nonfinite.check(dtype, d, 1, n, w, **kw)


@pytest.mark.parametrize("d,softcap,pairs,dtype,coarse,noref", masked.CASES_M)
def test_tiles_of_the_masked_layout(d, softcap, pairs, dtype, coarse, noref):
    wl = workloads.Workload("insm", 96, 8, 8, 2, 520 + d // 4, d, dtype, 8, 3, 48, softcap=50.0 if softcap else 0.0, mixture=4)
    inst.run_case(wl, pairs, big_norms=not noref)


@pytest.mark.parametrize("w", [40, 690])
@pytest.mark.parametrize("dtype,d,kw", [("bf16", 128, {}), ("f16", 80, dict(K=16, topk=3)), ("bf16", 64, dict(causal=False)), ("f16", 256, {}),
                                        ("bf16", 96, dict(pair_set=focus.FOCUS_PAIRS_SHARED))])
def test_values_that_are_not_finite_in_tiles(dtype, d, w, kw):
    nonfinite.check(dtype, d, 12, 700, w, **kw)


@pytest.mark.parametrize("size", ["high", "low"])
def test_range_of_halves_in_tiles(size, monkeypatch):
    f16_range.test_probabilities_outside_the_range_of_halves((1, 12, 4, 2100, 256, 4, 2, 200, True, 0.0), size, None, monkeypatch)


def test_rows_with_large_norms_in_tiles():
    """Disallowed keys with the largest logits must not move the row's reference (see test_gpu_masked)."""
    wl = workloads.Workload("m", 331, 45, 2, 1, 400, 64, "bf16", 4, 1, 16)
    inp = workloads.make_inputs(wl, "cuda")
    inp["q"] *= 8.0
    inp["k"] *= 8.0
    got, ref = harness.run_gpu(wl, inp), harness.run_gpu(wl, inp, vector=True)
    # one bf16 ulp of the output (2^-8 relative, values up to 4); the sum of probabilities that are each rounded by at most
    # 2^-9 of themselves is off by at most that factor, its logarithm by 2^-9, and logits of a few hundred by fp32 rounding
    assert (got["out"].float() - ref["out"].float()).abs().max() <= 2e-2
    assert ((got["lse"] - ref["lse"]).abs() <= 2.0 ** -9 + 1e-4 * ref["lse"].abs()).all()


@pytest.mark.parametrize("d,dtype,cap", [(64, "bf16", 50.0), (80, "f16", 30.0), (128, "f16", 50.0), (256, "bf16", 5.0)])
def test_softcap_of_single_pairs_keeps_32_bits(d, dtype, cap):
    """Rows that attend only their own key: lse is the capped logit, from a product whose sum is exact (halves of small whole numbers).
    The quotient, tanh (5 units in the last place at most), the product with the cap and the way to log2 units and back, two
    roundings each, are 12 roundings of 2^-24 relative; the one probability is 1."""
    wl = workloads.Workload("sc", 503, 2, 8, 4, 90, d, dtype, 32, 1, 1, softcap=cap)
    inp = workloads.make_inputs(wl, "cuda")
    for x in ("q", "k"):
        inp[x] = (inp[x].float() * 2.0).round().clamp(-4, 4).mul(0.5).to(inp[x].dtype)
    res = harness.run_gpu(wl, inp, scale=0.125)
    alone = (res["row_pairs"] == 1).cpu()
    logit = (inp["q"].double() * inp["k"].double().repeat_interleave(2, dim=1)).sum(-1).cpu() * 0.125
    want = cap * torch.tanh(logit / cap)
    assert alone.sum() > 100 and want[alone].abs().max() > 1.0
    assert ((res["lse"].cpu().double() - want)[alone].abs() <= 12 * 2.0 ** -24 * want[alone].abs()).all()


# about the limits of the launch choice, on either side of them
@pytest.mark.parametrize("B,Hq,n,d,causal", [(7, 8, 512, 64, True), (8, 8, 512, 64, True), (15, 8, 250, 256, True), (5, 1, 4096, 256, True), (5, 8, 500, 256, True),
                                             (14, 8, 256, 80, False), (5, 8, 512, 96, False), (5, 4, 512, 256, False), (11, 8, 250, 256, False), (1, 12, 512, 64, True)])
def test_softcap_given_to_the_attention_alone(B, Hq, n, d, causal):
    """The bucketing does not read the softcap: parameters without one prepare the same workspace."""
    wl = workloads.Workload("sk", 504, B, Hq, max(1, Hq // 4), n, d, "bf16", 4, 2, 60, causal=causal, softcap=30.0)
    inp = workloads.make_inputs(wl, "cuda")
    want = harness.run_gpu(wl, inp)
    p, plain = (focus.make_params(B, Hq, wl.Hkv, n, d, 4, 2, 60, causal=causal, softcap=cap) for cap in (30.0, 0.0))
    ws = focus.alloc_workspace(p)
    out, lse = torch.full_like(inp["q"], float("nan")), torch.empty_like(want["lse"])
    focus.focus_assign(plain, inp["q"], inp["k"], inp["centroids"], ws)
    focus.focus_attn_fwd(p, inp["q"], inp["k"], inp["v"], ws, out, lse)
    torch.cuda.synchronize()
    assert torch.equal(out, want["out"]) and torch.equal(lse, want["lse"])
