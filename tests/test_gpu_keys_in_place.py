"""The tiled kernel on keys that are read in place (masked layouts and the soft gate up to 8192 tokens): the last rows of the last key
tile, strided keys, the length where the copy begins, and the largest key norm found with the scores or by the scatter launch
(memberships given per token), which decides between the two forms of the softmax; against the vector kernel."""
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
