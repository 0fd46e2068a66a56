"""Logits whose exponentials leave the range of IEEE halves (2^-24 .. 2^16): the tiled kernel on float16 inputs, in every layout and
form, against the fp32 vector kernel."""
import pytest
import torch

from paper_2604_03260_amd import focus
from tests import harness

pytestmark = pytest.mark.gpu

SHAPES = [   # B, Hq, Hkv, n, d, K, topk, window, causal, softcap
    (2, 8, 8, 3000, 64, 4, 2, 256, True, 0.0), (2, 8, 4, 3001, 80, 16, 3, 100, True, 0.0), (1, 16, 4, 2500, 96, 8, 2, 2500, True, 0.0),
    (1, 16, 4, 2500, 128, 8, 1, 300, False, 0.0), (2, 8, 8, 3000, 128, 4, 2, 256, True, 50.0), (1, 4, 2, 2100, 256, 4, 2, 200, True, 0.0),
    (1, 4, 2, 20000, 64, 4, 2, 256, True, 0.0), (1, 2, 1, 18000, 128, 8, 1, 1000, True, 0.0), (1, 3, 1, 6000, 64, 4, 3, 700, False, 0.0),
    (1, 2, 2, 300, 64, 4, 2, 64, True, 0.0)]


def problem(shape, size):
    B, Hq, Hkv, n, d, K, topk, w, causal, softcap = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(n + d)
    if size == "high":               # a token is its own best key: up to 2^40, with rows of the same tile below and above 2^16
        k = torch.randn((B, Hkv, n, d), generator=g, device="cuda")
        scale = 8.0 + 18.0 * torch.rand((B, Hq, n, 1), generator=g, device="cuda")
        q = k.repeat_interleave(Hq // Hkv, 1)
        q = q * (scale * d ** 0.5 / q.norm(dim=-1, keepdim=True) ** 2)
    else:                            # every key of a head is far from every query: all of them around 2^-26
        u = torch.nn.functional.normalize(torch.randn((1, Hkv, 1, d), generator=g, device="cuda"), dim=-1)
        k = 0.3 * torch.randn((B, Hkv, n, d), generator=g, device="cuda") + 6.0 * u
        q = -3.0 * d ** 0.5 * u.repeat_interleave(Hq // Hkv, 1) + 0.2 * torch.randn((B, Hq, n, d), generator=g, device="cuda")
    v = torch.randn((B, Hkv, n, d), generator=g, device="cuda")
    c = torch.randn((Hkv, K, d), generator=g, device="cuda")
    p = focus.make_params(B, Hq, Hkv, n, d, K, topk, w, causal=causal, dtype="f16", softcap=softcap)
    q, k, v = q.half(), k.half(), v.half()
    ws = focus.alloc_workspace(p)
    focus.focus_assign(p, q, k, c, ws)
    return p, q, k, v, ws


def check(got, ref, lse, lse_ref):
    t = harness.TOL["f16"]
    # the queries times scale * log2(e) are rounded once more, 2^-12 of a component: of a logit of 26 over d >= 64 random
    # components 26 * 2^-12 / 8, far inside the tolerances
    assert torch.isfinite(got.float()).all()
    assert (got.float() - ref.float()).abs().max().item() <= t["out_max"]
    assert (got.float() - ref.float()).abs().mean().item() <= t["out_mean"]
    some = torch.isfinite(lse_ref)
    assert torch.equal(torch.isfinite(lse), some)
    assert (lse[some] - lse_ref[some]).abs().max().item() <= 4 * t["lse"]


@pytest.mark.parametrize("force", [None, "0", "1"])          # the chosen layout, class tiles, two passes
@pytest.mark.parametrize("size", ["high", "low"])
@pytest.mark.parametrize("shape", SHAPES)
def test_probabilities_outside_the_range_of_halves(shape, size, force, monkeypatch):
    if force is not None:
        monkeypatch.setenv("FOCUS_TWO_PASS", force)
    p, q, k, v, ws = problem(shape, size)
    got, ref = torch.empty_like(q), torch.empty_like(q)
    lse, lse_ref = (torch.empty(q.shape[:3], dtype=torch.float32, device="cuda") for _ in range(2))
    pairs, pairs_ref = (torch.empty(q.shape[:3], dtype=torch.int32, device="cuda") for _ in range(2))
    focus.focus_attn_fwd(p, q, k, v, ws, got, lse, pairs)
    focus.focus_attn_fwd(p, q, k, v, ws, ref, lse_ref, pairs_ref, vector=True)
    torch.cuda.synchronize()
    check(got, ref, lse, lse_ref)
    assert torch.equal(pairs, pairs_ref)


@pytest.mark.parametrize("size", ["high", "low"])
@pytest.mark.parametrize("shape", [s for s in SHAPES if s[7] < s[3]][:2] + [SHAPES[6]])
def test_restricted_sets(shape, size):
    """Rows without a pair in a set (a sum of zero) are rows of zeros, whatever the bound says."""
    p, q, k, v, ws = problem(shape, size)
    got, ref, parts = torch.empty_like(q), torch.empty_like(q), torch.empty((2,) + tuple(q.shape), dtype=q.dtype, device="cuda")
    lse, lse_ref = (torch.empty(q.shape[:3], dtype=torch.float32, device="cuda") for _ in range(2))
    part_lse = torch.empty((2,) + tuple(q.shape[:3]), dtype=torch.float32, device="cuda")
    focus.focus_attn_fwd_two_call(p, q, k, v, ws, got, lse, parts, part_lse)
    focus.focus_attn_fwd(p, q, k, v, ws, ref, lse_ref, vector=True)
    torch.cuda.synchronize()
    check(got, ref, lse, lse_ref)
