"""Infinities and NaN among the values: they reach the rows that attend their key, in their own component, as the
product with a positive probability gives it, and nothing else."""
import numpy as np
import pytest
import torch

from paper_2604_03260_amd import focus, workloads
from tests import harness

pytestmark = pytest.mark.gpu

INF, NAN = float("inf"), float("nan")


def _run(wl, inp, pair_set, vector):
    p = harness.params_of(wl)
    ws = focus.alloc_workspace(p)
    focus.focus_assign(p, inp["q"], inp["k"], inp["centroids"], ws)
    out = torch.empty_like(inp["q"])
    lse = torch.empty((wl.B, wl.Hq, wl.n), dtype=torch.float32, device="cuda")
    rp = torch.empty((wl.B, wl.Hq, wl.n), dtype=torch.int32, device="cuda")
    if vector:
        focus.focus_attn_fwd(p, inp["q"], inp["k"], inp["v"], ws, out, lse, rp, vector=True)
    else:
        focus.focus_attn_fwd_set(p, pair_set, inp["q"], inp["k"], inp["v"], ws, out, lse, rp)
    torch.cuda.synchronize()
    return dict(out=out, lse=lse, row_pairs=rp, views=focus.focus_workspace_views(p, ws))


def check(dtype, d, B, n, w, causal=True, softcap=0.0, pair_set=focus.FOCUS_PAIRS_ALL, K=8, topk=1, vector=False):
    wl = workloads.Workload("nf", 380, B, 4, 2, n, d, dtype, K, topk, w, causal=causal, softcap=softcap, mixture=3)
    inp = workloads.make_inputs(wl, "cuda")
    # alone in its component; two in one key; both signs in one component; twice the same
    bad = [(3, 7 % d, NAN), (100, 20, INF), (101, d - 1, -INF), (333, 5, INF), (333, 6, -INF), (420, 5, -INF), (500, 20, INF),
           (n - 1, 0, NAN), (n // 2, d // 2, INF)]
    bad = [(j, c, x) for j, c, x in bad if j < n]
    inp["v"][0, 0, [j for j, _, _ in bad], [c for _, c, _ in bad]] = 0.0
    clean = _run(wl, inp, pair_set, vector)
    mq, mk = harness.check_assign(wl, inp, clean)
    if pair_set == focus.FOCUS_PAIRS_ALL:
        harness.check_attn(wl, inp, clean, mq, mk)
    for j, c, x in bad:
        inp["v"][0, 0, j, c] = x
    got = _run(wl, inp, pair_set, vector)
    add = torch.zeros((wl.B, wl.Hq, n, d), device="cuda")
    i = np.arange(n)
    for h in range(wl.Hq // wl.Hkv):                  # the query heads of KV head 0
        for j, c, x in bad:
            dist = i - j
            cz = dist >= 0 if causal else np.ones(n, bool)
            loc = cz & (np.abs(dist) < w)
            share = cz & ((mq[0, h] & mk[0, 0, j]) != 0)
            at = {focus.FOCUS_PAIRS_ALL: share | loc, focus.FOCUS_PAIRS_SHARED: share, focus.FOCUS_PAIRS_CROSS_LOCAL: loc & ~share}[pair_set]
            add[0, h, torch.from_numpy(np.flatnonzero(at)).cuda(), c] += x
    spoiled = ~torch.isfinite(add)
    assert spoiled.sum() > 20 and (~spoiled[0, :2]).any(dim=-1).all()
    # everything else to the bit as with zeros in their place
    assert torch.equal(got["out"][~spoiled], clean["out"][~spoiled])
    assert torch.equal(got["lse"], clean["lse"]) and torch.equal(got["row_pairs"], clean["row_pairs"])
    o, e = got["out"][spoiled].float(), add[spoiled]
    assert torch.equal(torch.isnan(o), torch.isnan(e))
    assert torch.equal(o[~torch.isnan(o)], e[~torch.isnan(e)])


# a window inside a key tile, one that leaves whole tiles without a test, nearly everything
@pytest.mark.parametrize("w", [40, 300, 690])
@pytest.mark.parametrize("dtype,d,B,kw", [
    ("bf16", 128, 6, {}), ("f16", 80, 6, {}), ("bf16", 96, 6, dict(softcap=30.0)), ("bf16", 64, 8, dict(causal=False)), ("f16", 256, 1, {}),
    ("bf16", 128, 6, dict(pair_set=focus.FOCUS_PAIRS_SHARED, K=16, topk=3)), ("bf16", 64, 8, dict(pair_set=focus.FOCUS_PAIRS_CROSS_LOCAL))])
def test_masked_tiles(dtype, d, B, w, kw):
    check(dtype, d, B, 700, w, **kw)


# the kernel for a few work-groups of 32 rows: masked and dense layouts (a window past the end), one and two keys' worth
# of rows past a unit
@pytest.mark.parametrize("n,w", [(700, 40), (700, 300), (545, 544), (642, 5000), (130, 20)])
@pytest.mark.parametrize("dtype,d,kw", [("bf16", 64, {}), ("f16", 80, {}), ("bf16", 96, dict(softcap=30.0)), ("f16", 128, {}),
                                        ("bf16", 128, dict(causal=False)), ("f16", 64, dict(K=16, topk=3))])
def test_short_sequences(dtype, d, n, w, kw):
    check(dtype, d, 1, n, w, **kw)


# fp32: every head dim (those above 96 hold a quarter of a unit's values at a time), both numbers of wavefronts
@pytest.mark.parametrize("n,w", [(700, 40), (700, 300), (642, 5000)])
@pytest.mark.parametrize("d,B,kw", [(64, 1, {}), (64, 8, dict(causal=False)), (80, 1, dict(softcap=20.0)), (96, 6, {}), (128, 1, {}),
                                    (256, 1, {}), (256, 1, dict(causal=False, K=16, topk=3))])
def test_f32(d, B, n, w, kw):
    check("f32", d, B, n, w, **kw)


@pytest.mark.parametrize("tiles", [None, "0"])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128), ("f16", 80), ("bf16", 256)])
def test_vector_kernel(dtype, d, tiles, monkeypatch):
    """The masked layout and tiles of one class (where a tile's rows differ in what they attend)."""
    if tiles:
        monkeypatch.setenv("FOCUS_TWO_PASS", tiles)
    check(dtype, d, 1, 600, 90, vector=True)
