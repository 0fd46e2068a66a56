"""How a decode launch shares the walk out (16-bit caches): around whole rounds of 32 keys per share, shares that are resolved in two
passes, the change from even shares to chunks (128 heads), fewer entries than the launch was made for (list walks, a position
far below the capacity), against attention in float64 over the state's own memberships."""
import pytest
import torch

from paper_2604_03260_amd import focus
from tests import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,n,d,K,topk,w,dtype,at", [
    (1, 2, 1, 129, 64, 4, 2, 16, "bf16", None), (1, 2, 1, 128, 80, 4, 2, 16, "f16", None), (1, 20, 1, 4001, 96, 8, 2, 300, "bf16", None),
    (1, 8, 8, 2047, 128, 4, 2, 100, "f16", None), (1, 8, 8, 2049, 128, 16, 1, 100, "bf16", None),
    (1, 8, 8, 49153, 64, 4, 2, 100, "bf16", None), (2, 4, 4, 3000, 256, 8, 1, 64, "f16", None),
    (8, 16, 16, 4641, 64, 4, 2, 64, "bf16", None), (8, 16, 16, 4641, 64, 16, 1, 64, "bf16", None),
    (3, 43, 43, 2000, 64, 4, 2, 64, "f16", None), (3, 43, 43, 2000, 80, 32, 1, 20, "bf16", None),
    (1, 8, 8, 20000, 128, 4, 2, 300, "bf16", 700), (2, 6, 3, 9000, 96, 8, 1, 300, "f16", 31),
    (3, 43, 43, 6000, 64, 4, 2, 300, "bf16", 1000), (11, 12, 12, 5000, 80, 16, 1, 40, "f16", 1289), (33, 8, 4, 3000, 128, 8, 2, 3000, "bf16", 63)])
def test_shares_cover_the_walk_once(B, Hq, Hkv, n, d, K, topk, w, dtype, at):
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    g = torch.Generator(device="cuda")
    g.manual_seed(n + d)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").to(dt)
    kc, vc = rand(B, Hkv, n, d), rand(B, Hkv, n, d)
    c = torch.randn((Hkv, K, d), generator=g, device="cuda")
    p = focus.make_params(B, Hq, Hkv, n, d, K, topk, w, dtype=dtype)
    state = focus.alloc_decode_state(p)
    pos = n - 1 if at is None else at
    focus.focus_decode_prefill(p, pos, kc, c, state)
    q, k, v = rand(B, Hq, d), rand(B, Hkv, d), rand(B, Hkv, d)
    out, lse = torch.empty_like(q), torch.empty((B, Hq), dtype=torch.float32, device="cuda")
    pairs = torch.empty((B, Hq), dtype=torch.int32, device="cuda")
    if at is None:
        focus.focus_decode_step(p, pos, q, k, v, c, kc, vc, state, out, lse, pairs)
    else:
        pos_dev = torch.full((B,), pos, dtype=torch.int32, device="cuda")
        focus.focus_decode_step_at(p, pos_dev, q, k, v, c, kc, vc, state, out, lse, pairs)
    torch.cuda.synchronize()
    views = focus.focus_decode_state_views(p, state)
    m, G = pos + 1, Hq // Hkv
    for b in range(B):
        for h in range(Hq):
            x = (kc[b, h // G, :m].double() @ q[b, h].double()) / d ** 0.5
            row = (views["mk"][b, h // G, :m] & views["mq"][b, h]) != 0
            row[max(0, m - w):] = True
            assert pairs[b, h].item() == int(row.sum())              # every key once: no share left out or met twice
            x = x.masked_fill(~row, -float("inf"))
            ref = torch.softmax(x, 0) @ vc[b, h // G, :m].double()
            # probabilities and result are rounded to the 16-bit type: an average over `row.sum()` keys of N(0,1) values
            assert (out[b, h].double() - ref).abs().max() <= harness.TOL[dtype]["out_max"] * max(0.05, 4 / float(row.sum()) ** 0.5)
            assert (lse[b, h].double() - torch.logsumexp(x, 0)).abs() <= harness.TOL[dtype]["lse"]


@pytest.mark.parametrize("B,Hkv,K,topk,at,host", [(3, 43, 16, 1, 9000, True), (4, 40, 32, 1, 8999, True), (4, 40, 32, 1, 3000, True),
                                                  (8, 16, 16, 1, 9000, True), (3, 43, 4, 2, 1000, False), (3, 43, 4, 2, 6, False)])
def test_shares_of_a_walk(B, Hkv, K, topk, at, host):
    """How many work-groups share a walk.  Above 128 rows, where it is shorter than the launch knew (lists), a share is at least four
    rounds of 32 entries, one for each wavefront, unless there are eight shares or fewer; otherwise every round may be one.
    Partials without a key hold a maximum of -inf."""
    n, d, w = 9001, 64, 64
    g = torch.Generator(device="cuda")
    g.manual_seed(at)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    kc, vc, c = rand(B, Hkv, n, d), rand(B, Hkv, n, d), torch.randn((Hkv, K, d), generator=g, device="cuda")
    p = focus.make_params(B, Hkv, Hkv, n, d, K, topk, w)
    state = focus.alloc_decode_state(p)
    focus.focus_decode_prefill(p, at, kc, c, state)
    q, k, v = rand(B, Hkv, d), rand(B, Hkv, d), rand(B, Hkv, d)
    out = torch.empty_like(q)
    max_parts = min((n + 127) // 128, 384)
    used = B * Hkv * max_parts * (d + 4) * 4                     # the partials are the last block of the state
    parts = state[-((used + 255) // 256 * 256):][:used].view(torch.float32).view(B * Hkv, max_parts, d + 4)
    parts[:, :, d] = -float("inf")
    if host:
        focus.focus_decode_step(p, at, q, k, v, c, kc, vc, state, out)
    else:
        focus.focus_decode_step_at(p, torch.full((B,), at, dtype=torch.int32, device="cuda"), q, k, v, c, kc, vc, state, out)
    torch.cuda.synchronize()
    views = focus.focus_decode_state_views(p, state)
    lo = max(0, at - w + 1)                                      # first position of the window
    below = ((views["mk"][:, :, :lo] & views["mq"].view(B, Hkv, 1)) != 0).sum(-1)
    walk = torch.where(below >= lo, at + 1, at + 1 - lo + below) if topk == 1 else torch.full_like(below, at + 1)
    units = (walk.view(-1) + 31) // 32
    most = torch.clamp((units + 3) // 4, min=8) if host and B * Hkv > 128 else units
    live = (parts[:, :, d] > -float("inf")).sum(-1)
    assert bool((live >= 1).all()) and bool((live <= most).all()), (live.max().item(), most.min().item())
