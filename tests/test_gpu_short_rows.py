"""Bucketing of short rows in one launch: around whole wavefronts of 64 tokens, both work-group sizes (512 and 1024 tokens), group
counts at the edges of the scoring products (4, 8, 16 groups), strided views, scores that are not numbers."""
import numpy as np
import pytest
import torch

from paper_2604_03260_amd import focus, workloads
from tests import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 63, 65, 511, 512, 513, 1024])
@pytest.mark.parametrize("K,topk,dtype,d", [(4, 1, "bf16", 64), (3, 1, "f32", 64), (8, 3, "f16", 64), (5, 2, "f32", 64), (16, 2, "bf16", 96),
                                            (9, 4, "f32", 128), (8, 2, "bf16", 128), (4, 2, "f32", 256)])
def test_short_rows_are_exact(n, K, topk, dtype, d):
    wl = workloads.Workload("sr", 400 + n, 1, 4, 2, n, d, dtype, K, topk, max(1, min(n - 1, 40)), mixture=3)
    inp = workloads.make_inputs(wl, "cuda")
    if n > 64:                                        # a token without numbers takes the first topk groups
        inp["k"][0, 1, 64] = float("nan")
        inp["v"][0, 1, 64] = 0.0
    res = harness.run_gpu(wl, inp)
    mq, mk = harness.check_assign(wl, inp, res)
    if n <= 64:
        harness.check_attn(wl, inp, res, mq, mk)
    harness.check_pair_totals(wl, res, mq, mk)


@pytest.mark.parametrize("B,n,K,topk,d", [(43, 448, 4, 2, 64), (43, 449, 4, 2, 64), (43, 512, 8, 1, 64), (171, 130, 16, 2, 64), (170, 256, 9, 2, 80)])
def test_many_short_rows_are_exact(B, n, K, topk, d):
    """Where a launch of many rows changes from one work-group per row to sort blocks (512 and 2048 rows; 32 bits)."""
    wl = workloads.Workload("mr", 900 + n, B, 8, 4, n, d, "f32", K, topk, 33, mixture=3)
    inp = workloads.make_inputs(wl, "cuda")
    res = harness.run_gpu(wl, inp)
    mq, mk = harness.check_assign(wl, inp, res)
    harness.check_pair_totals(wl, res, mq, mk)


def test_short_rows_through_strides():
    B, Hq, Hkv, n, d = 2, 4, 2, 200, 64
    x = torch.randn((B, n, Hq + 2 * Hkv, d), device="cuda").to(torch.bfloat16)
    q, k, v = (y.permute(0, 2, 1, 3) for y in (x[:, :, :Hq], x[:, :, Hq:Hq + Hkv], x[:, :, Hq + Hkv:]))
    c = torch.randn((Hkv, 6, d), device="cuda")
    got = []
    for contiguous in (False, True):
        t = [y.contiguous() if contiguous else y for y in (q, k, v)]
        out = torch.empty((B, Hq, n, d), dtype=x.dtype, device="cuda")
        p = focus.make_params(B, Hq, Hkv, n, d, 6, 2, 20, q_strides=focus.strides_of(t[0]), kv_strides=focus.strides_of(t[1]))
        ws = focus.alloc_workspace(p)
        focus.focus_assign(p, t[0], t[1], c, ws)
        focus.focus_attn_fwd(p, t[0], t[1], t[2], ws, out)
        torch.cuda.synchronize()
        got.append([out.cpu()] + [y.cpu().clone() for y in focus.focus_workspace_views(p, ws).values()])
    for a, b in zip(*got):
        assert np.array_equal(a.view(torch.int16).numpy() if a.dtype == torch.bfloat16 else a.numpy(),
                              b.view(torch.int16).numpy() if b.dtype == torch.bfloat16 else b.numpy())
