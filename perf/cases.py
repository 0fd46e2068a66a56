"""What is measured: the calls a program makes of this library, each through its public entry points.

Kinds of case
  prefill   focus_assign + focus_attn_fwd: one layer of a prompt (membership, bucketing, attention).
  route     focus_route + focus_assign_tokens: the per-layer router and the bucketing of its memberships.
  decode    focus_decode_prefill + `steps` x focus_decode_step (or focus_decode_step_at): one layer of a
            generation call that takes over a cached context and produces `steps` tokens per sequence.
  soft      focus_attn_soft_fwd: one layer of the training forward with the soft gate.

Inputs follow the recipe of the package's workloads: q, k, v ~ N(0,1), with `mixture` clusters a mean per
(tensor, head, cluster) ~ N(0, 0.5^2) and Zipf cluster weights, rounded to the storage type; centroids ~ N(0,1)
with unit rows.
"""
import math

import torch

from paper_2604_03260_amd import focus

TORCH_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
DEVICE = "cuda"


def listed():
    prefill = dict(kind="prefill", causal=True, softcap=0.0, mixture=0, packed=False)
    decode = dict(kind="decode", softcap=0.0, mixture=0)
    return [
        # The shortest prompts, of a 12-head model with 64 components per head: launches and latency count.
        dict(prefill, name="prompt_512", dtype="bf16", B=1, Hq=12, Hkv=12, n=512, d=64, K=4, topk=2, window=128),
        # The same model kept in 32 bits (evaluation against a reference, small models).
        dict(prefill, name="prefill_f32_1k", dtype="f32", B=1, Hq=12, Hkv=12, n=1024, d=64, K=4, topk=2, window=128),
        # A batch of ordinary prompts, clustered tokens.
        dict(prefill, name="prefill_batch8_4k", dtype="bf16", B=8, Hq=12, Hkv=12, n=4096, d=64, K=4, topk=2,
             window=256, mixture=4),
        # Odd sizes and the wider options together: IEEE halves, 80 components, a ragged length, more membership
        # sets than exact classes, q, k, v as views of one packed projection.
        dict(prefill, name="prefill_f16_ragged", dtype="f16", B=3, Hq=15, Hkv=5, n=5003, d=80, K=16, topk=3,
             window=300, mixture=8, packed=True),
        # Grouped queries and a long prompt: the main prefill case.
        dict(prefill, name="prefill_32k", dtype="bf16", B=1, Hq=32, Hkv=8, n=32768, d=128, K=4, topk=2, window=1024),
        # 64 heads, eight groups, soft-capped logits, clustered tokens: where the mask is sparse.
        dict(prefill, name="prefill_softcap_128k", dtype="bf16", B=1, Hq=64, Hkv=8, n=131072, d=128, K=8, topk=1,
             window=4096, softcap=50.0, mixture=8),
        # The largest prompt that a pass of under two seconds allows.
        dict(prefill, name="prefill_256k", dtype="bf16", B=1, Hq=32, Hkv=8, n=262144, d=128, K=4, topk=2, window=4096),
        # The router of a layer with 4096 hidden components, ten Sinkhorn rounds, then the bucketing for all heads.
        dict(kind="route", name="route_32k", dtype="bf16", B=1, Hq=32, Hkv=8, n=32768, d=128, d_model=4096, d_g=16,
             K=4, topk=2, window=1024, sinkhorn=10, soft=False),
        # A batch of short generations that end one by one, positions in device memory.
        dict(decode, name="decode_batch8_4k", dtype="bf16", B=8, Hq=12, Hkv=12, ctx=4096, steps=32, d=64, K=4, topk=2,
             window=256, mixture=4, device_pos=True),
        # Generation after the main prompt length.
        dict(decode, name="decode_32k", dtype="bf16", B=1, Hq=32, Hkv=8, ctx=32768, steps=32, d=128, K=4, topk=2,
             window=1024, device_pos=False),
        # Generation after a long context, hard assignment, soft-capped logits.
        dict(decode, name="decode_softcap_128k", dtype="bf16", B=1, Hq=64, Hkv=8, ctx=131072, steps=16, d=128, K=8,
             topk=1, window=4096, softcap=50.0, mixture=8, device_pos=False),
        # A training forward of the soft gate.
        dict(kind="soft", name="soft_gate_8k", dtype="bf16", B=1, Hq=32, Hkv=8, n=8192, d=128, K=4, window=1024, lam=8.0),
    ]


# ---------------------------------------------------------------- more cases of the same ranges

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng):
    """(Hq, Hkv, d): multi-head and grouped layouts around 768 .. 8192 query components."""
    return rng.choice([(12, 12, 64), (16, 16, 64), (32, 8, 128), (64, 8, 128), (16, 4, 256), (40, 8, 96), (15, 5, 80),
                       (32, 32, 128), (24, 8, 128), (14, 2, 64)])


def _groups(rng):
    return rng.choice([(4, 1), (4, 2), (8, 1), (8, 2), (8, 3), (16, 2), (16, 3), (32, 2)])


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "prefill", "prefill", "route", "decode", "decode", "soft"])
    Hq, Hkv, d = _heads(rng)
    K, topk = _groups(rng)
    mixture = rng.choice([0, 0, 4, 8])
    if kind == "prefill":
        dtype = rng.choice(["bf16", "bf16", "bf16", "f16", "f32"])
        n = _log_int(rng, 200, 2048 if dtype == "f32" else 65536)
        B = rng.choice([1, 1, 2, 4, 8])
        # at most about the work of the largest listed case, and the 32-bit cases small as they are in use
        most = 2e9 if dtype == "f32" else 32 * 65536.0 ** 2
        while B > 1 and B * Hq * float(n) * n > most:
            B //= 2
        n = min(n, int(math.sqrt(most / (B * Hq))))
        return dict(kind=kind, dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, n=n, d=d, K=K, topk=topk,
                    window=max(1, min(n - 1, _log_int(rng, 64, 4096))), causal=rng.random() < 0.85,
                    softcap=rng.choice([0.0, 0.0, 0.0, 30.0, 50.0]), mixture=mixture, packed=rng.random() < 0.3)
    if kind == "route":
        n, B = _log_int(rng, 500, 131072), rng.choice([1, 1, 2, 4])
        n = max(500, n // B)
        return dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f16", "f32"]), B=B, Hq=Hq, Hkv=Hkv, n=n, d=d,
                    d_model=Hq * d, d_g=rng.choice([8, 16, 16, 16, 32]), K=K, topk=topk,
                    window=max(1, min(n - 1, _log_int(rng, 64, 4096))), sinkhorn=rng.choice([0, 10, 10]),
                    soft=rng.random() < 0.3)
    if kind == "decode":
        B = rng.choice([1, 1, 2, 8])
        ctx = max(300, _log_int(rng, 500, 131072) // B)
        return dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f16"]), B=B, Hq=Hq, Hkv=Hkv, ctx=ctx,
                    steps=rng.randint(8, 32), d=d, K=K, topk=topk, window=_log_int(rng, 64, 4096),
                    softcap=rng.choice([0.0, 0.0, 50.0]), mixture=mixture, device_pos=rng.random() < 0.4)
    d = rng.choice([64, 80, 96, 128])
    return dict(kind="soft", dtype=rng.choice(["bf16", "bf16", "f16"]), B=rng.choice([1, 2]), Hq=Hq, Hkv=Hkv,
                n=_log_int(rng, 300, 8192), d=d, K=rng.choice([4, 8, 16, 32]), window=_log_int(rng, 64, 1024),
                lam=rng.choice([2.0, 8.0]))


# ---------------------------------------------------------------- what a program has in hand before the call

def _generator(seed, salt):
    g = torch.Generator(device=DEVICE)
    g.manual_seed((int(seed) * 1000003 + salt) % (1 << 62))
    return g


def _fill(t, g, mixture, z):
    """t [B,H,n,d] (any strides) drawn head by head."""
    B, H, n, d = t.shape
    mu = torch.randn((H, mixture, d), generator=g, device=DEVICE) * 0.5 if mixture else None
    for b in range(B):
        for h in range(H):
            x = torch.randn((n, d), generator=g, device=DEVICE)
            if mixture:
                x += mu[h][z[b]]
            t[b, h] = x.to(t.dtype)


def _clusters(case, n, seed):
    if not case.get("mixture"):
        return None
    w = 1.0 / torch.arange(1, case["mixture"] + 1, device=DEVICE, dtype=torch.float32)
    return torch.multinomial(w.expand(case["B"], -1), n, replacement=True, generator=_generator(seed, 4))


def _centroids(Hkv, K, d, seed):
    c = torch.randn((Hkv, K, d), generator=_generator(seed, 3), device=DEVICE, dtype=torch.float64)
    return (c / c.norm(dim=-1, keepdim=True)).float().contiguous()


def _qkv(case, n, seed):
    """q [B,Hq,n,d], k, v [B,Hkv,n,d]; with `packed` they are views of one [B,n,(Hq+2Hkv)d] projection."""
    B, Hq, Hkv, d = case["B"], case["Hq"], case["Hkv"], case["d"]
    dt = TORCH_DTYPES[case["dtype"]]
    if case.get("packed"):
        x = torch.empty((B, n, Hq + 2 * Hkv, d), dtype=dt, device=DEVICE)
        q, k, v = (y.permute(0, 2, 1, 3) for y in (x[:, :, :Hq], x[:, :, Hq:Hq + Hkv], x[:, :, Hq + Hkv:]))
    else:
        q = torch.empty((B, Hq, n, d), dtype=dt, device=DEVICE)
        k = torch.empty((B, Hkv, n, d), dtype=dt, device=DEVICE)
        v = torch.empty_like(k)
    z = _clusters(case, n, seed)
    for salt, t in enumerate((q, k, v)):
        _fill(t, _generator(seed, salt), case.get("mixture", 0), z)
    return q, k, v


def _hidden(case, seed):
    """Hidden states, router projection and router centroids, as the package's router inputs."""
    B, n, dm, dg = case["B"], case["n"], case["d_model"], case["d_g"]
    hidden = torch.empty((B, n, dm), dtype=TORCH_DTYPES[case["dtype"]], device=DEVICE)
    g = _generator(seed, 7)
    rows = max(1, (1 << 24) // dm)
    for b in range(B):
        for r in range(0, n, rows):
            hidden[b, r:r + rows] = torch.randn((min(rows, n - r), dm), generator=g, device=DEVICE).to(hidden.dtype)
    w_g = (torch.randn((dm, dg), generator=_generator(seed, 8), device=DEVICE) / dm ** 0.5).contiguous()
    c = torch.randn((case["K"], dg), generator=_generator(seed, 9), device=DEVICE, dtype=torch.float64)
    return hidden, w_g, (c / c.norm(dim=-1, keepdim=True)).float().contiguous()


def _soft_assignment(case, seed):
    s = torch.randn((case["B"], case["n"], case["K"]), generator=_generator(seed, 11), device=DEVICE) * 3.0
    return torch.softmax(s, dim=-1).contiguous()


def _lengths(case, seed):
    """Tokens every sequence of a batch produces: between half of the steps and all of them."""
    x = torch.rand((case["B"],), generator=_generator(seed, 12), device=DEVICE).tolist()
    return [max(1, int(round(case["steps"] * (0.5 + 0.5 * u)))) for u in x]


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind}
    if kind == "prefill":
        B, Hq, Hkv, n, d = (case[x] for x in ("B", "Hq", "Hkv", "n", "d"))
        q, k, v = _qkv(case, n, seed)
        if case["packed"]:
            s["out"] = torch.empty((B, n, Hq, d), dtype=q.dtype, device=DEVICE)
            out = s["out"].permute(0, 2, 1, 3)
            strides = dict(q_strides=focus.strides_of(q), kv_strides=focus.strides_of(k), o_strides=focus.strides_of(out))
        else:
            s["out"] = out = torch.empty_like(q)
            strides = {}
        p = focus.make_params(B, Hq, Hkv, n, d, case["K"], case["topk"], case["window"], causal=case["causal"],
                              dtype=case["dtype"], softcap=case["softcap"], **strides)
        s.update(p=p, q=q, k=k, v=v, o=out, c=_centroids(Hkv, case["K"], d, seed), ws=focus.alloc_workspace(p),
                 lse=torch.empty((B, Hq, n), dtype=torch.float32, device=DEVICE))
        s["views"] = focus.focus_workspace_views(p, s["ws"])
    elif kind == "route":
        B, Hq, Hkv, n, d = (case[x] for x in ("B", "Hq", "Hkv", "n", "d"))
        s["hidden"], s["w_g"], s["rc"] = _hidden(case, seed)
        s["rp"] = focus.make_route_params(B, n, case["d_model"], case["d_g"], case["K"], case["topk"], dtype=case["dtype"],
                                          sinkhorn_iters=case["sinkhorn"], tau=0.1)
        s["rws"] = focus.alloc_route_workspace(s["rp"])
        s["masks"] = torch.empty((B, n), dtype=torch.int32, device=DEVICE)
        s["soft"] = torch.empty((B, n, case["K"]), dtype=torch.float64, device=DEVICE) if case["soft"] else None
        s["k"] = torch.empty((B, Hkv, n, d), dtype=TORCH_DTYPES[case["dtype"]], device=DEVICE)
        _fill(s["k"], _generator(seed, 1), 0, None)
        s["p"] = focus.make_params(B, Hq, Hkv, n, d, case["K"], case["topk"], case["window"], dtype=case["dtype"])
        s["ws"] = focus.alloc_workspace(s["p"])
        s["views"] = focus.focus_workspace_views(s["p"], s["ws"])
    elif kind == "decode":
        B, Hq, Hkv, d, T = (case[x] for x in ("B", "Hq", "Hkv", "d", "steps"))
        n = case["ctx"] + T
        q, kc, vc = _qkv(dict(case, Hq=Hkv), n, seed)       # the caches; their last rows are overwritten by the steps
        del q
        dt = kc.dtype
        new = {"q": torch.empty((T, B, Hq, d), dtype=dt, device=DEVICE)}
        new["k"] = torch.empty((T, B, Hkv, d), dtype=dt, device=DEVICE)
        new["v"] = torch.empty_like(new["k"])
        for salt, t in ((20, new["q"]), (21, new["k"]), (22, new["v"])):
            t.copy_(torch.randn(t.shape, generator=_generator(seed, salt), device=DEVICE))
        p = focus.make_params(B, Hq, Hkv, n, d, case["K"], case["topk"], case["window"], dtype=case["dtype"],
                              softcap=case["softcap"])
        s.update(p=p, n_ctx=case["ctx"], kc=kc, vc=vc, c=_centroids(Hkv, case["K"], d, seed),
                 state=focus.alloc_decode_state(p).zero_(), T=T)
        s["out"] = torch.empty((T, B, Hq, d), dtype=dt, device=DEVICE)
        s["lse"] = torch.empty((T, B, Hq), dtype=torch.float32, device=DEVICE)
        s["pos"] = None
        s["rows"] = [(new["q"][t], new["k"][t], new["v"][t], s["out"][t], s["lse"][t]) for t in range(T)]
        s["views"] = focus.focus_decode_state_views(p, s["state"])
        if case["device_pos"]:
            # positions in device memory, advanced between the steps; a sequence that has produced all its tokens
            # (between half and all of the steps) leaves the batch: its position is outside the caches
            ends = _lengths(case, seed)
            s["pos"] = [torch.tensor([case["ctx"] + t if t < e else -1 for e in ends], dtype=torch.int32, device=DEVICE)
                        for t in range(T)]
            s["out"].zero_()
            s["lse"].zero_()
    else:
        q, k, v = _qkv(case, case["n"], seed)
        p = focus.make_params(case["B"], case["Hq"], case["Hkv"], case["n"], case["d"], case["K"], 1, case["window"],
                              dtype=case["dtype"])
        s.update(p=p, q=q, k=k, v=v, g=_soft_assignment(case, seed), lam=case["lam"], ws=focus.alloc_soft_workspace(p),
                 out=torch.empty_like(q), lse=torch.empty((case["B"], case["Hq"], case["n"]), dtype=torch.float32, device=DEVICE))
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    kind = s["kind"]
    if kind == "prefill":
        focus.focus_assign(s["p"], s["q"], s["k"], s["c"], s["ws"])
        focus.focus_attn_fwd(s["p"], s["q"], s["k"], s["v"], s["ws"], s["o"], s["lse"])
        return {"out": s["out"], "lse": s["lse"], "membership": s["views"]}
    if kind == "route":
        focus.focus_route(s["rp"], s["hidden"], s["w_g"], s["rc"], s["rws"], s["masks"], s["soft"])
        focus.focus_assign_tokens(s["p"], s["masks"], s["k"], s["ws"])
        return {"masks": s["masks"], "soft": s["soft"], "membership": s["views"]}
    if kind == "decode":
        focus.focus_decode_prefill(s["p"], s["n_ctx"], s["kc"], s["c"], s["state"])
        for t, (q, k, v, out, lse) in enumerate(s["rows"]):
            if s["pos"] is not None:
                focus.focus_decode_step_at(s["p"], s["pos"][t], q, k, v, s["c"], s["kc"], s["vc"], s["state"], out, lse)
            else:
                focus.focus_decode_step(s["p"], s["n_ctx"] + t, q, k, v, s["c"], s["kc"], s["vc"], s["state"], out, lse)
        return {"out": s["out"], "lse": s["lse"], "mk": s["views"]["mk"], "counts": s["views"]["counts"]}
    focus.focus_attn_soft_fwd(s["p"], s["lam"], s["g"], s["q"], s["k"], s["v"], s["ws"], s["out"], s["lse"])
    return {"out": s["out"], "lse": s["lse"]}


# ---------------------------------------------------------------- what a pass cannot do without

def _share(K, k):
    """P(two uniform k-subsets of K groups have a group in common)."""
    none = 1.0
    for i in range(k):
        none *= max(0.0, (K - k - i) / (K - i))
    return 1.0 - none


def work(case):
    el = 4 if case["dtype"] == "f32" else 2
    kind, B, Hq, Hkv, d, K = (case[x] for x in ("kind", "B", "Hq", "Hkv", "d", "K"))
    if kind in ("prefill", "route"):
        n, w, k = case["n"], min(case["window"], case["n"]), case["topk"]
        lists = (Hq + Hkv) * B * n * 4.0 * (1 + k)                  # memberships and group lists
    if kind == "prefill":
        share = _share(K, k)
        if case["causal"]:
            local = w * (n - (w - 1) / 2.0)
            pairs = local + share * (n * (n + 1) / 2.0 - local)
        else:
            local = min(float(n) * n, (2 * w - 1) * float(n) - w * (w - 1.0))
            pairs = local + share * (float(n) * n - local)
        return {"bytes": B * n * d * el * (2.0 * Hq + 2 * Hkv) + lists + B * Hq * n * 4.0, "flops": 4.0 * d * B * Hq * pairs}
    if kind == "route":
        dm, dg = case["d_model"], case["d_g"]
        return {"bytes": B * n * dm * el + dm * dg * 4.0 + lists + B * n * 4.0 + (B * n * K * 8.0 if case["soft"] else 0.0),
                "flops": B * n * dg * 2.0 * (dm + K)}
    if kind == "decode":
        G, w, ctx, T = Hq // Hkv, min(case["window"], case["ctx"]), case["ctx"], case["steps"]
        below = (ctx - w) * (1.0 - (1.0 - _share(K, case["topk"])) ** G)        # keys some head of the KV head attends
        one = (ctx - w) * _share(K, case["topk"]) + w
        alive = 0.75 if case["device_pos"] else 1.0
        return {"bytes": B * Hkv * ctx * (d * el + 4.0) + alive * T * B * Hkv * (w + below) * 2.0 * d * el,
                "flops": alive * T * B * Hq * one * 4.0 * d}
    n = case["n"]
    return {"bytes": B * n * d * el * (2.0 * Hq + 2 * Hkv) + B * n * K * 4.0 + B * Hq * n * 4.0,
            "flops": B * Hq * n * (n + 1) / 2.0 * (4.0 * d + 2.0 * K)}


# ---------------------------------------------------------------- how far apart two correct results may be

def tolerance(case):
    """Whole numbers (memberships, lists, counts) are the same.  Attention in 16-bit types: the probabilities and the
    result are rounded to the type (2^-9, 2^-12), and so may the scaled queries be; in 32 bits the sums' order.
    Seen against 64 bits: 1.7e-3 .. 2.7e-3, 2.1e-4 .. 2.5e-4, 2.8e-7 .. 4.9e-7; the router's scores 7e-16."""
    if case["kind"] == "route":
        return {"rel": 1e-9}            # what the tests of the router hold the normalised scores to
    return {"rel": {"bf16": 1e-2, "f16": 1.2e-3, "f32": 2e-6}[case["dtype"]]}


# ---------------------------------------------------------------- the same in 64 bits

def _membership(x, c, topk):
    """Bit masks [B,H,n] of the topk best centroids of every row (ties to the smaller group)."""
    s = torch.matmul(x.double(), c.double().transpose(-1, -2).contiguous())
    top = torch.sort(s, dim=-1, descending=True, stable=True).indices[..., :topk]
    return (1 << top).sum(-1)


def _softmax_rows(q, k, v, allowed, scale, softcap, gate=None):
    """(out, lse) of one block of rows in float64; `allowed` [rows, keys], `gate` multiplies the logits."""
    x = q.double() @ k.double().t().contiguous() * scale
    if gate is not None:
        x *= gate
    if softcap:
        x = softcap * torch.tanh(x / softcap)
    x.masked_fill_(~allowed, -math.inf)
    lse = torch.logsumexp(x, dim=-1)
    return torch.exp_(x.sub_(lse[:, None])) @ v.double(), lse


def exact(case, seed):
    kind, B, Hq, Hkv, d = (case[x] for x in ("kind", "B", "Hq", "Hkv", "d"))
    if kind in ("prefill", "soft"):
        if float(B) * Hq * case["n"] ** 2 > 4e10:
            return None
        return _exact_prefill(case, prepare(case, seed))
    if kind == "route":
        return _exact_route(case, prepare(case, seed)) if case["soft"] else None
    return _exact_decode(case, prepare(case, seed))


def _exact_prefill(case, s):
    B, Hq, Hkv, n, d = (case[x] for x in ("B", "Hq", "Hkv", "n", "d"))
    w, scale, soft = case["window"], 1.0 / math.sqrt(d), case["kind"] == "soft"
    causal, cap = case.get("causal", True), case.get("softcap", 0.0)
    out = torch.empty((B, Hq, n, d), dtype=torch.float64, device=DEVICE)
    lse = torch.empty((B, Hq, n), dtype=torch.float64, device=DEVICE)
    j = torch.arange(n, device=DEVICE)
    rows = max(64, min(n, (1 << 26) // n))
    for h in range(Hq):
        hk = h // (Hq // Hkv)
        for b in range(B):
            if not soft:
                mq = _membership(s["q"][b, h], s["c"][hk], case["topk"])
                mk = _membership(s["k"][b, hk], s["c"][hk], case["topk"])
            for r in range(0, n, rows):
                i = j[r:r + rows, None]
                m = min(n, r + rows) if causal else n
                dist = i - j[None, :m]
                local = (dist < w) if causal else (dist.abs() < w)
                gate = None
                if soft:
                    ok = dist >= 0
                    aff = torch.sigmoid(case["lam"] * (s["g"][b, r:r + rows].double() @ s["g"][b, :m].double().t().contiguous()))
                    gate = torch.where(local, torch.ones_like(aff), aff)
                else:
                    ok = local | ((mq[r:r + rows, None] & mk[None, :m]) != 0)
                    if causal:
                        ok &= dist >= 0
                out[b, h, r:r + rows], lse[b, h, r:r + rows] = _softmax_rows(
                    s["q"][b, h, r:r + rows], s["k"][b, hk, :m], s["v"][b, hk, :m], ok, scale, cap, gate)
    if case.get("packed"):
        out = out.permute(0, 2, 1, 3).contiguous()
    if soft:
        return {"out": out, "lse": lse}
    return {"out": out, "lse": lse, "membership": {name: None for name in s["views"]}}


def _exact_route(case, s):
    soft = torch.empty((case["B"], case["n"], case["K"]), dtype=torch.float64, device=DEVICE)
    for b in range(case["B"]):
        z = torch.cat([x.double() @ s["w_g"].double() for x in s["hidden"][b].split(4096)])
        x = z @ s["rc"].double().t().contiguous()
        if case["sinkhorn"] == 0:
            soft[b] = x / 0.1
            continue
        Q = torch.exp((x - x.max()) / 0.1)
        for _ in range(case["sinkhorn"]):
            Q = Q / Q.sum(0, keepdim=True)
            Q = Q / Q.sum(1, keepdim=True)
        soft[b] = Q
    return {"masks": None, "soft": soft, "membership": {name: None for name in s["views"]}}


def _exact_decode(case, s):
    B, Hq, Hkv, d, T, ctx = (case[x] for x in ("B", "Hq", "Hkv", "d", "steps", "ctx"))
    scale, cap, G = 1.0 / math.sqrt(d), case["softcap"], Hq // Hkv
    out = torch.zeros((T, B, Hq, d), dtype=torch.float64, device=DEVICE)
    lse = torch.zeros((T, B, Hq), dtype=torch.float64, device=DEVICE)
    for b in range(B):
        for hk in range(Hkv):
            k, v = s["kc"][b, hk].clone(), s["vc"][b, hk].clone()
            for t in range(T):
                k[ctx + t], v[ctx + t] = s["rows"][t][1][b, hk], s["rows"][t][2][b, hk]
            mk = _membership(k, s["c"][hk], case["topk"])
            q = torch.stack([s["rows"][t][0][b, hk * G:(hk + 1) * G] for t in range(T)]).reshape(T * G, d)
            mq = _membership(q, s["c"][hk], case["topk"])
            i = (ctx + torch.arange(T, device=DEVICE)).repeat_interleave(G)[:, None]
            dist = i - torch.arange(ctx + T, device=DEVICE)[None, :]
            ok = (dist >= 0) & ((dist < case["window"]) | ((mq[:, None] & mk[None, :]) != 0))
            o, l = _softmax_rows(q, k, v, ok, scale, cap)
            out[:, b, hk * G:(hk + 1) * G], lse[:, b, hk * G:(hk + 1) * G] = o.reshape(T, G, d), l.reshape(T, G)
    if s["pos"] is not None:
        for t in range(T):
            done = s["pos"][t] < 0
            out[t, done], lse[t, done] = 0.0, 0.0
    return {"out": out, "lse": lse, "mk": None, "counts": None}
