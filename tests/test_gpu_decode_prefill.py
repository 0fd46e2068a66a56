"""The cache state that focus_decode_prefill builds (masks, lists, counts, window pointers through the next steps) at the
edges of its scoring tiles (16 and 64 keys, 128-byte row chunks) and list chunks (2048 positions, 8 groups)."""
import numpy as np
import pytest
import torch

from oracle import focus_oracle as fo
from paper_2604_03260_amd import focus, workloads
from tests import harness

pytestmark = pytest.mark.gpu


def _check_state(v, mk, n_ctx):
    got = v["mk"].cpu().numpy().view(np.uint32)[:, :, :n_ctx]
    assert np.array_equal(got, mk)
    lists, counts = v["lists"].cpu().numpy(), v["counts"].cpu().numpy()
    B, Hkv, K = counts.shape
    for b in range(B):
        for h in range(Hkv):
            for g in range(K):
                want = np.flatnonzero((mk[b, h] >> g) & 1)
                assert counts[b, h, g] == len(want)
                assert np.array_equal(lists[b, h, g, :len(want)], want)


@pytest.mark.parametrize("n_ctx", [1, 15, 17, 63, 65, 257, 2047, 2049, 4100])
@pytest.mark.parametrize("d,K,topk,dtype,window", [
    (64, 4, 2, "bf16", 100), (80, 9, 2, "f16", 1), (96, 16, 3, "bf16", 2049), (128, 8, 1, "f32", 5000), (256, 32, 4, "bf16", 17)])
def test_prefilled_state_is_exact(n_ctx, d, K, topk, dtype, window):
    wl = workloads.Workload("dp", 370 + K, 1, 4, 2, n_ctx, d, dtype, K, topk, window, mixture=3)
    inp = workloads.make_inputs(wl, "cuda")
    n = n_ctx + 3
    kc = torch.zeros((1, 2, n, d), dtype=inp["k"].dtype, device="cuda")
    vc = torch.zeros_like(kc)
    kc[:, :, :n_ctx], vc[:, :, :n_ctx] = inp["k"], inp["v"]
    p = focus.make_params(1, 4, 2, n, d, K, topk, window, dtype=dtype)
    pb = fo.Problem(1, 4, 2, n_ctx, d, K, topk, window, dtype=dtype)
    mk = fo.membership(pb, workloads.to_host_bits(inp["k"]), inp["centroids"].cpu().numpy(), False)
    state = focus.alloc_decode_state(p)
    focus.focus_decode_prefill(p, n_ctx, kc, inp["centroids"], state)
    torch.cuda.synchronize()
    _check_state(focus.focus_decode_state_views(p, state), mk, n_ctx)
    # the window pointers: two steps, their pair counts against the masks
    for t in range(2):
        pos = n_ctx + t
        g = torch.Generator(device="cuda")
        g.manual_seed(pos)
        q, k, v = (torch.randn((1, h, d), generator=g, device="cuda").to(kc.dtype) for h in (4, 2, 2))
        out, pairs = torch.empty_like(q), torch.empty((1, 4), dtype=torch.int32, device="cuda")
        focus.focus_decode_step(p, pos, q, k, v, inp["centroids"], kc, vc, state, out, None, pairs)
        torch.cuda.synchronize()
        views = focus.focus_decode_state_views(p, state)
        allk = views["mk"].cpu().numpy().view(np.uint32)[0, :, :pos + 1]
        mq = views["mq"].cpu().numpy().view(np.uint32)[0]
        for h in range(4):
            row = (allk[h // 2] & mq[h]) != 0
            row[max(0, pos - window + 1):] = True
            assert pairs[0, h].item() == int(row.sum())


def test_prefill_from_token_masks_is_exact():
    n_ctx, K, topk = 4099, 32, 2
    rng = np.random.default_rng(5)
    masks = np.zeros((2, n_ctx), np.uint32)
    for b in range(2):
        for i in range(n_ctx):
            masks[b, i] = np.bitwise_or.reduce(1 << rng.choice(K, topk, replace=False).astype(np.uint32))
    p = focus.make_params(2, 2, 1, n_ctx + 5, 64, K, topk, 64)
    state = focus.alloc_decode_state(p)
    focus.focus_decode_prefill_tokens(p, n_ctx, torch.from_numpy(masks.view(np.int32)).cuda(), state)
    torch.cuda.synchronize()
    _check_state(focus.focus_decode_state_views(p, state), masks[:, None, :], n_ctx)


@pytest.mark.parametrize("d,dtype,K,topk", [(64, "bf16", 4, 2), (80, "f16", 8, 1), (96, "bf16", 8, 2), (128, "f16", 4, 2)])
def test_step_with_rows_of_the_next_round_in_flight(d, dtype, K, topk):
    """Launches of about 430 work-groups of 512-entry chunks (the longest ones, with two work-groups on most compute units):
    a ragged last chunk, scan and list walks, against attention in float64 over the state's own memberships."""
    B, Hq, Hkv, n = 1, 16, 8, 27000 + d
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").to(dt)
    kc, vc = rand(B, Hkv, n, d), rand(B, Hkv, n, d)
    c = torch.randn((Hkv, K, d), generator=g, device="cuda")
    p = focus.make_params(B, Hq, Hkv, n, d, K, topk, 700, dtype=dtype)
    state = focus.alloc_decode_state(p)
    focus.focus_decode_prefill(p, n - 1, kc, c, state)
    q, k, v = rand(B, Hq, d), rand(B, Hkv, d), rand(B, Hkv, d)
    out, lse = torch.empty_like(q), torch.empty((B, Hq), dtype=torch.float32, device="cuda")
    focus.focus_decode_step(p, n - 1, q, k, v, c, kc, vc, state, out, lse)
    torch.cuda.synchronize()
    views = focus.focus_decode_state_views(p, state)
    for h in range(Hq):
        x = (kc[0, h // 2].double() @ q[0, h].double()) / d ** 0.5
        row = (views["mk"][0, h // 2] & views["mq"][0, h]) != 0
        row[n - 700:] = True
        x = x.masked_fill(~row, -float("inf"))
        ref = torch.softmax(x, 0) @ vc[0, h // 2].double()
        # an average of thousands of rows: the tolerances of the 16-bit types scaled to its size (outputs near 0.02)
        assert (out[0, h].double() - ref).abs().max() <= harness.TOL[dtype]["out_max"] * 0.05
        assert (lse[0, h].double() - torch.logsumexp(x, 0)).abs() <= harness.TOL[dtype]["lse"]
