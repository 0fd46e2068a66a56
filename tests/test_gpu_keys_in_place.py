"""The tiled kernel on keys that are read in place (masked layouts and the soft gate up to 8192 tokens): strided keys, the length where
the copy begins, keys of the last, ragged tile that decide their rows, keys that are not finite, and the largest key norm found
with the scores or by the scatter launch (memberships given per token), which decides between the two forms of the softmax;
against the vector kernel."""
import pytest
import torch

from paper_2604_03260_amd import focus
from tests import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens", [False, True])
@pytest.mark.parametrize("big", [1.0, 12.0])              # 12: logits past the bound of the form without a reference
@pytest.mark.parametrize("n,d,K,topk,dtype,causal,packed", [
    (4225, 64, 4, 2, "bf16", True, False), (4290, 80, 16, 3, "f16", True, True), (2100, 128, 8, 4, "bf16", False, True),
    (8191, 96, 32, 2, "bf16", True, False), (8192, 64, 16, 2, "f16", True, False), (8193, 64, 16, 2, "bf16", True, False)])
def test_keys_in_place(n, d, K, topk, dtype, causal, packed, big, tokens):
    B, Hq, Hkv = 1, 6, 3
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    g = torch.Generator(device="cuda")
    g.manual_seed(n + d)
    x = torch.randn((B, n, Hq + 2 * Hkv, d), generator=g, device="cuda")
    x[:, n // 2, Hq:Hq + Hkv] *= big * d ** 0.5 / 4         # one key decides the bound
    x = x.to(dt)
    q, k, v = (y.permute(0, 2, 1, 3) for y in (x[:, :, :Hq], x[:, :, Hq:Hq + Hkv], x[:, :, Hq + Hkv:]))
    if not packed:
        q, k, v = q.contiguous(), k.contiguous(), v.contiguous()
    c = torch.randn((Hkv, K, d), generator=g, device="cuda")
    p = focus.make_params(B, Hq, Hkv, n, d, K, topk, 200, causal=causal, dtype=dtype, q_strides=focus.strides_of(q),
                          kv_strides=focus.strides_of(k))
    ws = focus.alloc_workspace(p)
    ws.fill_(0xee)                                          # nothing may be read before it is written
    if tokens:
        perm = torch.rand((B, n, K), generator=g, device="cuda").argsort(-1)[..., :topk]
        masks = (1 << perm).sum(-1).to(torch.int32)
        focus.focus_assign_tokens(p, masks, k, ws)
    else:
        focus.focus_assign(p, q, k, c, ws)
    got, ref = (torch.empty((B, Hq, n, d), dtype=dt, device="cuda") for _ in range(2))
    lse, lse_ref = (torch.empty((B, Hq, n), dtype=torch.float32, device="cuda") for _ in range(2))
    focus.focus_attn_fwd(p, q, k, v, ws, got, lse)
    focus.focus_attn_fwd(p, q, k, v, ws, ref, lse_ref, vector=True)
    torch.cuda.synchronize()
    t = harness.TOL[dtype]
    # a logit carries the rounding of a query row (one half ulp of the type) times its size: up to |q||k|/sqrt(d) of the big key
    size = max(1.0, big * d ** 0.5 / 4)
    assert (got.float() - ref.float()).abs().max().item() <= t["out_max"] * size
    assert (got.float() - ref.float()).abs().mean().item() <= t["out_mean"]
    assert (lse - lse_ref).abs().max().item() <= t["lse"] * size


@pytest.mark.parametrize("n,d,dtype,packed,soft", [
    (4225, 64, "bf16", True, False), (4225, 64, "bf16", False, False), (4290, 80, "f16", True, False), (4259, 96, "f16", False, False),
    (4287, 128, "bf16", True, False), (2177, 256, "bf16", True, False), (4225, 128, "bf16", True, True), (1089, 64, "f16", True, True), (190, 80, "bf16", False, True)])
def test_the_last_tile_holds_its_own_keys(n, d, dtype, packed, soft):
    """The last n % 64 rows each meet one key, their own, that outweighs all others, with a value of its own: a row of the last tile
    read from anywhere else is another result."""
    B, Hq, Hkv, tail = 2, 6, 3, n % 64
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    g = torch.Generator(device="cuda")
    g.manual_seed(n + d)
    x = 0.1 * torch.randn((B, n, Hq + 2 * Hkv, d), generator=g, device="cuda")
    own = torch.randn((B, tail, Hkv, d), generator=g, device="cuda")
    own *= 16.0 / own.norm(dim=-1, keepdim=True)
    x[:, n - tail:, Hq:Hq + Hkv] = own                      # q.k / sqrt(d) = 256 / sqrt(d) >= 16 with itself
    x[:, n - tail:, :Hq] = own.repeat_interleave(Hq // Hkv, 2)
    x[:, n - tail:, Hq + Hkv:] *= 20.0
    x = x.to(dt)
    q, k, v = (y.permute(0, 2, 1, 3) for y in (x[:, :, :Hq], x[:, :, Hq:Hq + Hkv], x[:, :, Hq + Hkv:]))
    if not packed:
        q, k, v = q.contiguous(), k.contiguous(), v.contiguous()
    strides = dict(q_strides=focus.strides_of(q), kv_strides=focus.strides_of(k))
    out = torch.empty((B, Hq, n, d), dtype=dt, device="cuda")
    if soft:
        p = focus.make_params(B, Hq, Hkv, n, d, 4, 1, 100, dtype=dtype, **strides)
        ws = focus.alloc_soft_workspace(p)
        ws.fill_(0xee)
        gates = torch.softmax(torch.randn((B, n, 4), generator=g, device="cuda"), -1).contiguous()
        focus.focus_attn_soft_fwd(p, 8.0, gates, q, k, v, ws, out)
    else:
        c = torch.randn((Hkv, 8, d), generator=g, device="cuda")
        p = focus.make_params(B, Hq, Hkv, n, d, 8, 3, 100, dtype=dtype, **strides)
        ws = focus.alloc_workspace(p)
        ws.fill_(0xee)
        focus.focus_assign(p, q, k, c, ws)
        focus.focus_attn_fwd(p, q, k, v, ws, out)
    torch.cuda.synchronize()
    want = v[:, :, n - tail:].repeat_interleave(Hq // Hkv, 1).float()
    got = out[:, :, n - tail:].float()
    # the others: n keys of logits within +-2 and values of 0.1, and up to 63 of the tail that are orthogonal up to 6 / sqrt(d) of
    # their size: together below 1 % of e^16 for every d here; the result is rounded to its type
    assert (got - want).abs().max().item() <= 0.02 * want.abs().max().item()


@pytest.mark.parametrize("tokens", [False, True])
@pytest.mark.parametrize("bad", ["nan", "inf"])
@pytest.mark.parametrize("n,d,K,topk,dtype", [(4225, 64, 4, 2, "bf16"), (4290, 80, 16, 3, "f16"), (2500, 128, 8, 4, "bf16")])
def test_keys_that_are_not_finite(n, d, K, topk, dtype, bad, tokens):
    """Only the rows that attend such a key may follow it: the norm that is not finite rules the form without a reference out."""
    B, Hq, Hkv = 1, 6, 3
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k, v = (torch.randn((B, h, n, d), generator=g, device="cuda").to(dt) for h in (Hq, Hkv, Hkv))
    k[0, 1, n // 3, 5] = float(bad)
    k[0, 2, n - 1, 0] = float(bad)
    c = torch.randn((Hkv, K, d), generator=g, device="cuda")
    p = focus.make_params(B, Hq, Hkv, n, d, K, topk, 200, dtype=dtype)
    ws = focus.alloc_workspace(p)
    ws.fill_(0xee)
    if tokens:
        perm = torch.rand((B, n, K), generator=g, device="cuda").argsort(-1)[..., :topk]
        focus.focus_assign_tokens(p, (1 << perm).sum(-1).to(torch.int32), k, ws)
    else:
        focus.focus_assign(p, q, k, c, ws)
    got, ref = torch.empty_like(q), torch.empty_like(q)
    focus.focus_attn_fwd(p, q, k, v, ws, got)
    focus.focus_attn_fwd(p, q, k, v, ws, ref, vector=True)
    views = focus.focus_workspace_views(p, ws)
    torch.cuda.synchronize()
    i = torch.arange(n, device="cuda")
    for h in range(Hq):
        hit = torch.zeros(n, dtype=torch.bool, device="cuda")
        for hk, j in ((1, n // 3), (2, n - 1)):
            if h // 2 == hk:
                hit |= (i >= j) & ((i - j < 200) | ((views["mq"][0, h] & views["mk"][0, hk, j]) != 0))
        assert torch.isfinite(got[0, h][~hit]).all()
        assert (got[0, h][~hit].float() - ref[0, h][~hit].float()).abs().max().item() <= harness.TOL[dtype]["out_max"]
        if bad == "nan":
            assert torch.isnan(got[0, h][hit]).all()
