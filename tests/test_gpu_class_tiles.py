"""Class-ordered tiles, one pass (FOCUS_TWO_PASS=0), on the shapes that the size estimate gives to the masked layout, and
the forms of the bucketing and of the fp32 kernel that only large or widely strided problems take.  Every test states
the layout it means, so that another choice of layout cannot leave it without its subject."""
import numpy as np
import pytest
import torch

from paper_2604_03260_amd import focus, workloads
from tests import harness
from tests import test_gpu_graph, test_gpu_parity, test_gpu_strides, test_gpu_two_call, test_layout_choice

pytestmark = pytest.mark.gpu


def layout_of(wl, monkeypatch):
    return test_layout_choice.layout_of(harness.params_of(wl), monkeypatch)


def is_dense(wl):
    return wl.window >= wl.n or 2 * wl.topk > wl.K


# ---------------------------------------------------------------- tests of other files, over class tiles

@pytest.mark.parametrize("case", test_gpu_two_call.CASES, ids=[str(i) for i in range(len(test_gpu_two_call.CASES))])
def test_restricted_sets(case, monkeypatch):
    """Sets A and B, exact and coarse classes, causal or not, every type (the fp32 kernel included)."""
    B, Hq, Hkv, n, d, dtype, K, topk, w, cap = case[:10]
    wl = workloads.Workload("t", 70, B, Hq, Hkv, n, d, dtype, K, topk, w, causal=case[10] if len(case) > 10 else True, softcap=cap)
    if not is_dense(wl):
        assert layout_of(wl, monkeypatch) == "masked"     # what tests/test_gpu_two_call.py runs by itself
    monkeypatch.setenv("FOCUS_TWO_PASS", "0")
    test_gpu_two_call.test_sets_merge_and_two_call_small(case)


@pytest.mark.parametrize("kw", test_gpu_strides.CASES, ids=[str(i) for i in range(len(test_gpu_strides.CASES))])
def test_strided_tensors(kw, monkeypatch):
    monkeypatch.setenv("FOCUS_TWO_PASS", "0")
    test_gpu_strides.test_strided_tensors_give_the_contiguous_result(kw)


@pytest.mark.parametrize("wl", test_gpu_parity.SMALL_CASES, ids=[w.name for w in test_gpu_parity.SMALL_CASES])
def test_small_cases(wl, monkeypatch):
    monkeypatch.setenv("FOCUS_TWO_PASS", "0")
    test_gpu_parity.test_small_cases_all_rows(wl)


@pytest.mark.parametrize("name", ["test_noncausal_mid_size_sampled_rows", "test_coarse_classes_mid_size_sampled_rows"])
def test_mid_sizes(name, monkeypatch):
    monkeypatch.setenv("FOCUS_TWO_PASS", "0")
    getattr(test_gpu_parity, name)()


def test_coarse_classes_at_32768_tokens(monkeypatch):
    monkeypatch.setenv("FOCUS_TWO_PASS", "0")
    test_gpu_parity.test_cfg3_variants_full_sampled_rows("k32_top2_coarse")


def test_coarse_classes_that_the_estimate_chooses(monkeypatch):
    wl = workloads.Workload("coarse_long", 390, 1, 2, 1, 300000 + 91, 64, "bf16", 32, 2, 700, mixture=8)
    assert layout_of(wl, monkeypatch) == "one pass"
    inp = workloads.make_inputs(wl, "cuda")
    res = harness.run_gpu(wl, inp)
    mq, mk = harness.check_assign(wl, inp, res)
    harness.check_attn(wl, inp, res, mq, mk, rows=workloads.sample_rows(wl, 128))


@pytest.mark.parametrize("kw", [dict(dtype="bf16", d=128), dict(dtype="f16", d=96, K=8, topk=2), dict(dtype="f32", d=64),
                                dict(dtype="bf16", d=128, K=32, topk=2)])
def test_graph_replay(kw, monkeypatch):
    monkeypatch.setenv("FOCUS_TWO_PASS", "0")
    test_gpu_graph.test_assign_and_attention_replay_from_a_graph(kw)


# ---------------------------------------------------------------- masked layouts whose histograms need the scan launch

@pytest.mark.parametrize("K,topk,n,dtype", [(32, 2, 40000, "bf16"), (16, 3, 66001, "f16"), (32, 3, 33100, "f32")])
def test_masked_layout_with_the_scan_launch(K, topk, n, dtype, monkeypatch):
    """More than 4096 entries of group histograms per row: ceil(n / 256) * K."""
    wl = workloads.Workload("scan", 391, 1, 2, 1, n, 64, dtype, K, topk, 300, mixture=8)
    assert layout_of(wl, monkeypatch) == "masked" and -(-n // 256) * K > 4096
    inp = workloads.make_inputs(wl, "cuda")
    res = harness.run_gpu(wl, inp)
    mq, mk = harness.check_assign(wl, inp, res)
    rows = workloads.sample_rows(wl, 192)
    harness.check_attn(wl, inp, res, mq, mk, rows=rows)
    harness.check_pair_totals(wl, res, mq, mk)
    # memberships given per token take the same scan and scatter
    p = harness.params_of(wl)
    ws = focus.alloc_workspace(p)
    out = torch.empty_like(inp["q"])
    masks = torch.from_numpy(mk[:, 0].astype(np.uint32).view(np.int32).copy()).cuda()
    focus.focus_assign_tokens(p, masks, inp["k"], ws)
    focus.focus_attn_fwd(p, inp["q"], inp["k"], inp["v"], ws, out)
    torch.cuda.synchronize()
    both = np.repeat(mk[:, :1], wl.Hq, axis=1)
    res2 = dict(out=out, lse=None, row_pairs=None, views=focus.focus_workspace_views(p, ws))
    assert np.array_equal(res2["views"]["mq"].cpu().numpy().view(np.uint32), both)
    harness.check_attn(wl, inp, res2, both, mk, rows=rows)


# ---------------------------------------------------------------- key and value rows far apart

def far_apart(x, pitch):
    """A copy of x [1,H,n,d] whose rows lie `pitch` elements apart, heads side by side between them."""
    _, H, n, d = x.shape
    buf = torch.empty(((n - 1) * pitch + H * d,), dtype=x.dtype, device="cuda")
    y = buf.as_strided((1, H, n, d), (H * d, d, pitch, 1))
    y.copy_(x)
    return y


# row pitches of 16 MiB and more, and of less where the last row still lies 4 GiB past the first
@pytest.mark.parametrize("tiles", [None, "0"])
@pytest.mark.parametrize("dtype,d,K,topk,mib,n", [
    ("f32", 64, 8, 2, 16, 290), ("f32", 80, 8, 2, 17, 270), ("f32", 96, 16, 3, 16, 260), ("f32", 128, 8, 1, 9, 480),
    ("f32", 256, 4, 1, 16, 270), ("bf16", 64, 8, 2, 16, 290), ("f16", 128, 8, 1, 9, 480)])
def test_rows_far_apart(dtype, d, K, topk, mib, n, tiles, monkeypatch):
    wl = workloads.Workload("far", 392, 1, 4, 2, n, d, dtype, K, topk, 33, mixture=3)
    assert layout_of(wl, monkeypatch) == "masked"
    if tiles:
        monkeypatch.setenv("FOCUS_TWO_PASS", tiles)
    inp = workloads.make_inputs(wl, "cuda")
    pitch = (mib << 20) // inp["k"].element_size()
    k, v = far_apart(inp["k"], pitch), far_apart(inp["v"], pitch)
    strides = (2 * d, d, pitch)
    p = focus.make_params(1, 4, 2, n, d, K, topk, 33, dtype=dtype, kv_strides=strides)
    ws = focus.alloc_workspace(p)
    out = torch.empty_like(inp["q"])
    lse = torch.empty((1, 4, n), dtype=torch.float32, device="cuda")
    rp = torch.empty((1, 4, n), dtype=torch.int32, device="cuda")
    focus.focus_assign(p, inp["q"], k, inp["centroids"], ws)
    focus.focus_attn_fwd(p, inp["q"], k, v, ws, out, lse, rp)
    torch.cuda.synchronize()
    res = dict(out=out, lse=lse, row_pairs=rp, views=focus.focus_workspace_views(p, ws))
    mq, mk = harness.check_assign(wl, inp, res)
    harness.check_attn(wl, inp, res, mq, mk)
    harness.check_pair_totals(wl, res, mq, mk)
