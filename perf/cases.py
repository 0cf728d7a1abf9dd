"""The performance cases of the library: the calls a serving engine and its trainer make.

A speculative-decoding rollout engine runs, per step, the decoder layers over the 1+k
positions of every sequence, the LM head and the accept rule; per turn of an agent, a prefill
of the new window behind a cached context; and the actor scores the emitted tokens with the
recorded routes. The cases are those calls through the public binding, single layers and
blocks first (each with a tolerance of its own), and three whole calls that return logits.

Shapes are the 35B-A3B-like mixture of experts of workloads.py (d 2048, 32 query / 4 kv heads
x 128, 128 experts top-8, FFN 768, vocabulary 151936, 16-token KV blocks) and its tiny f32
decoder. Inputs are random with seeded generators on the GPU: weights N(0, 0.02^2) (fp8
experts quantised per output channel), residual stream and KV cache N(0, 1), physical KV
blocks a random permutation, drafts drawn from a perturbed target. As with a trained router,
every row has K experts it clearly prefers (its row holds a multiple of their router rows), so
that no rounding changes a route; the sets are uniform, or skewed with the router bias.

Kinds of case:
  layer    decoder_forward of one layer on B sequences of 1+k new positions (k = n - 1: a
           prefill window of n positions) at contexts ctx_lo..ctx_hi
  prefill  the whole prefill call (embedding, two layers, LM head of the last rows)
  score    the whole recompute call with replayed routes (embedding, two layers, LM head of
           every row, log-probs)
  moe      moe_layer on normalised rows
  accept   spec_accept on given logits
"""
import math

import torch

import paper_2607_21653_amd as molt

BF16 = torch.bfloat16
BIG = dict(d=2048, Hq=32, Hkv=4, D=128, E=128, K=8, F=768, V=151936)
TINY = dict(d=256, Hq=4, Hkv=4, D=64, E=8, K=2, F=512, V=2048)
THETA, EPS, STD = 1.0e6, 1.0e-6, 0.02


def listed():
    return [
        # one agent decoding alone with 4 drafts: the smallest layer call, latency-bound
        dict(name="layer_one_sequence", kind="layer", B=1, k=4, ctx_lo=1500, ctx_hi=1500, experts="bf16", zipf=0.0),
        # speculation disabled (k = 0): plain decode of a ragged batch
        dict(name="layer_plain_decode", kind="layer", B=48, k=0, ctx_lo=300, ctx_hi=6000, experts="bf16", zipf=0.0),
        # an ordinary verify batch: the layer workload of workloads.py
        dict(name="layer_bf16", kind="layer", B=64, k=4, ctx_lo=4096, ctx_hi=4096, experts="bf16", zipf=0.0),
        # long, variable agent contexts: attention over the split key range
        dict(name="layer_long_ctx", kind="layer", B=16, k=4, ctx_lo=32768, ctx_hi=65536, experts="bf16", zipf=0.0),
        # fp8 experts under skewed load with 8 drafts: the largest verify batch
        dict(name="layer_fp8_zipf", kind="layer", B=256, k=8, ctx_lo=2048, ctx_hi=2048, experts="fp8", zipf=1.2),
        # first prompts of two agents: a fresh prefill window (compute-bound)
        dict(name="layer_prompt", kind="layer", B=2, k=1999, ctx_lo=0, ctx_hi=0, experts="bf16", zipf=0.0),
        # a tool result appended to a session whose history is cached: the whole prefill call
        dict(name="prefill_cache_hit", kind="prefill", B=1, n=256, ctx_lo=8192, ctx_hi=8192, experts="bf16"),
        # the expert block on its own, fp8 experts, an odd row count
        dict(name="moe_fp8", kind="moe", T=1003, experts="fp8", zipf=0.0),
        # the accept rule for one sequence: launch-bound
        dict(name="accept_one", kind="accept", B=1, k=4, V=151936, q=True),
        # the accept rule of a full verify batch
        dict(name="accept_batch", kind="accept", B=128, k=4, V=151936, q=True),
        # the actor's recompute of a full verify batch, routes replayed: a whole call
        dict(name="score_batch", kind="score", B=128, k=4, ctx_lo=8192, ctx_hi=8192, experts="bf16"),
        # the tiny f32 decoder (debugging and numerics runs): a whole call in f32
        dict(name="score_tiny_f32", kind="score", B=4, k=3, ctx_lo=64, ctx_hi=128, experts="f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "prompt", "prefill", "moe", "accept", "accept", "score", "score_f32"])
    if kind == "layer":
        B, k = _log(rng, 1, 256), rng.choice([0, 1, 2, 3, 4, 4, 5, 6, 7, 8])
        hi = max(16, min(65536, 1 << 20 if B == 1 else (1 << 20) // B))   # at most 2^20 cached tokens in all
        c = _log(rng, 16, hi)
        return dict(kind="layer", B=B, k=k, ctx_lo=rng.randint(c // 2, c), ctx_hi=c,
                    experts=rng.choice(["bf16", "fp8"]), zipf=rng.choice([0.0, 1.2]))
    if kind == "prompt":   # prefill windows, at most 4000 rows, fresh or behind a cached context
        B = _log(rng, 1, 16)
        c = rng.choice([0, _log(rng, 100, 8192)])
        return dict(kind="layer", B=B, k=_log(rng, 100, 4000 // B) - 1, ctx_lo=c // 2, ctx_hi=c,
                    experts=rng.choice(["bf16", "fp8"]), zipf=0.0)
    if kind == "prefill":
        B = _log(rng, 1, 4)
        c = _log(rng, 64, 8192)
        return dict(kind="prefill", B=B, n=_log(rng, 16, 512 // B), ctx_lo=c // 2, ctx_hi=c, experts="bf16")
    if kind == "moe":
        return dict(kind="moe", T=_log(rng, 1, 2500), experts=rng.choice(["bf16", "fp8"]), zipf=rng.choice([0.0, 1.2]))
    if kind == "accept":
        return dict(kind="accept", B=_log(rng, 1, 128), k=rng.randint(0, 4), V=_log(rng, 2000, 151936),
                    q=rng.choice([True, True, False]))
    c = _log(rng, 32, 2048)
    if kind == "score":
        return dict(kind="score", B=_log(rng, 1, 128), k=rng.randint(0, 4), ctx_lo=c // 2, ctx_hi=c, experts="bf16")
    return dict(kind="score", B=_log(rng, 1, 6), k=rng.randint(0, 3), ctx_lo=c // 16, ctx_hi=c // 8, experts="f32")


# ---------------------------------------------------------------------------- inputs

def _dims(case):
    return TINY if case["experts"] == "f32" else BIG


def _gen(seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + what * 7919 + 17) & ((1 << 62) - 1))
    return g


def _randn(g, shape, dtype, std=1.0):
    t = torch.randn(shape, generator=g, device="cuda", dtype=dtype)
    return t if std == 1.0 else t.mul_(std)


def _fp8(g, shape):
    w = _randn(g, shape, torch.float32, STD)
    s = w.abs().amax(-1) / 448.0
    return (w / s.unsqueeze(-1)).to(torch.float8_e4m3fn).view(torch.uint8), s


def _moe_weights(case, g):
    m = _dims(case)
    d, E, F = m["d"], m["E"], m["F"]
    dt = torch.float32 if case["experts"] == "f32" else BF16
    w = {"w_router": _randn(g, (E, d), dt, STD), "s_gate_up": None, "s_down": None, "router_bias": None}
    if case["experts"] == "fp8":
        w["w_gate_up"], w["s_gate_up"] = _fp8(g, (E, 2 * F, d))
        w["w_down"], w["s_down"] = _fp8(g, (E, d, F))
    else:
        w["w_gate_up"], w["w_down"] = _randn(g, (E, 2 * F, d), dt, STD), _randn(g, (E, d, F), dt, STD)
    if case.get("zipf"):
        rank = torch.randperm(E, generator=g, device="cuda").float() + 1.0
        w["router_bias"] = -case["zipf"] * rank.log()
    return w


def _prefer(case, g, n, w):
    """[n, d] f32: what n rows hold of the router rows of the K experts that each prefers, drawn
    uniformly or by the router's bias."""
    m = _dims(case)
    z = 0.9 * _randn(g, (n, m["E"]), torch.float32)
    if w["router_bias"] is not None:
        z += w["router_bias"]
    r = w["w_router"].float()
    pick = torch.zeros_like(z).scatter_(1, z.topk(m["K"], -1).indices, 11.0 if case.get("zipf") else 7.0)
    return pick @ (r / r.norm(dim=-1, keepdim=True))


def _layer_weights(case, g):
    m = _dims(case)
    d, D = m["d"], m["D"]
    dt = torch.float32 if case["experts"] == "f32" else BF16
    w = _moe_weights(case, g)
    for norm in ("attn_norm", "moe_norm"):
        w[norm] = 1.0 + _randn(g, (d,), torch.float32, 0.1)
    w["w_qkv"] = _randn(g, ((m["Hq"] + 2 * m["Hkv"]) * D, d), dt, STD)
    w["w_o"] = _randn(g, (d, m["Hq"] * D), dt, STD)
    return w


def _inputs(case, seed):
    """Row-major weights and inputs of a layer, prefill or score case."""
    m, B = _dims(case), case["B"]
    kp1 = case["n"] if case["kind"] == "prefill" else case["k"] + 1
    dt = torch.float32 if case["experts"] == "f32" else BF16
    L = 1 if case["kind"] == "layer" else 2
    g = _gen(seed, 1)
    s = {"kp1": kp1, "layers": [_layer_weights(case, g) for _ in range(L)]}
    # contexts spread evenly over their range, in random order
    ctx = case["ctx_lo"] + (torch.randperm(B, generator=g, device="cuda") * 2 + 1) * (
        case["ctx_hi"] - case["ctx_lo"]) // (2 * B)
    need = (ctx + kp1 + 15) // 16
    nb, mb = int(need.sum()), int(need.max())
    ids = torch.randperm(nb, generator=g, device="cuda").int()
    bt = torch.full((B, mb), -1, dtype=torch.int32, device="cuda")
    bt[torch.arange(mb, device="cuda")[None, :] < need[:, None]] = ids
    s["ctx"], s["bt"] = ctx.int(), bt
    s["kc"] = [_randn(g, (nb, m["Hkv"], 16, m["D"]), dt) for _ in range(L)]
    s["vc"] = [_randn(g, (nb, m["Hkv"], m["D"], 16), dt) for _ in range(L)]
    if case["kind"] == "layer":
        s["x"] = _randn(g, (B * kp1, m["d"]), torch.float32) + _prefer(case, g, B * kp1, s["layers"][0])
        return s
    embed = _randn(g, (m["V"], m["d"]), torch.float32)
    if case["kind"] == "prefill":
        for w in s["layers"]:
            embed += _prefer(case, g, m["V"], w)
    s["head"] = {"embed": embed.to(dt), "lm_head": _randn(g, (m["V"], m["d"]), dt, STD),
                 "final_norm": 1.0 + _randn(g, (m["d"],), torch.float32, 0.1)}
    s["tokens"] = torch.randint(0, m["V"], (B, kp1), generator=g, device="cuda").int()
    if case["kind"] == "prefill":
        s["lens"] = torch.randint(max(1, kp1 // 2), kp1 + 1, (B,), generator=g, device="cuda").int()
        return s
    s["targets"] = torch.randint(0, m["V"], (B, kp1), generator=g, device="cuda").int()
    s["routes"] = torch.rand((L, B * kp1, m["E"]), generator=g, device="cuda").topk(m["K"], -1).indices.int()
    return s


def _accept_inputs(case, seed):
    B, k, V = case["B"], case["k"], case["V"]
    g = _gen(seed, 2)
    logits = _randn(g, (B, k + 1, V), torch.float32, 2.0)
    q = torch.softmax(logits[:, :k] + 0.5 * _randn(g, (B, k, V), torch.float32), -1)
    drafts = torch.empty((B, k), dtype=torch.int32, device="cuda")
    for i in range(k):   # drafts are drawn from q (Gumbel-max)
        u = torch.rand((B, V), generator=g, device="cuda").clamp_(min=1e-30)
        drafts[:, i] = (q[:, i].log() - (-u.log()).log()).argmax(-1).int()
    s = {"logits": logits, "drafts": drafts, "u": torch.rand((B, k + 1), generator=g, device="cuda")}
    s["q"] = q.contiguous() if case["q"] and k > 0 else None
    return s


def _moe_inputs(case, seed):
    g = _gen(seed, 3)
    w = _moe_weights(case, g)
    return {"x": (_randn(g, (case["T"], BIG["d"]), torch.float32) + _prefer(case, g, case["T"], w)).to(BF16), "w": w}


def _model(case, s):
    m = _dims(case)
    return molt.Model(s["layers"], s.get("head"), n_q_heads=m["Hq"], n_kv_heads=m["Hkv"], head_dim=m["D"],
                      top_k=m["K"], rms_eps=EPS, rope_theta=THETA)


def _buffer(nbytes):
    return torch.empty(max(1, nbytes), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    if kind == "accept":
        s = _accept_inputs(case, seed)
        s["ws"] = _buffer(molt.load().molt_spec_accept_workspace_size(case["B"], case["k"], case["V"]))
    elif kind == "moe":
        s = _moe_inputs(case, seed)
        w = s["w"]
        for key in ("w_router", "w_gate_up", "w_down"):
            w[key] = molt.pack_weights(w[key])
        s["ws"] = _buffer(molt.load().molt_moe_layer_workspace_size(
            case["T"], BIG["d"], BIG["E"], BIG["K"], BIG["F"], molt.MOLT_BF16,
            molt.MOLT_FP8_E4M3 if case["experts"] == "fp8" else molt.MOLT_BF16))
    else:
        s = _inputs(case, seed)
        s["model"] = _model(case, s)
        s["kv"] = molt.KVCache(s["kc"], s["vc"], s["bt"], s["ctx"])
        mb = s["bt"].shape[1]
        if kind == "layer":
            size = molt.decoder_workspace_size(s["model"], case["B"], case["k"], mb)
        elif kind == "prefill":
            size = molt.prefill_workspace_size(s["model"], case["B"], case["n"], mb)
        else:
            size = molt.score_tokens_workspace_size(s["model"], case["B"], case["k"], mb)
        del s["layers"]     # the model keeps its tiled copies
        s["ws"] = _buffer(size)
    s["case"] = case
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "accept":
        tokens, n, lp = molt.spec_accept(s["logits"], s["drafts"], s["u"], s["q"], workspace=s["ws"])
        return {"tokens": tokens, "n_accepted": n, "logprobs": lp}
    if kind == "moe":
        w = s["w"]
        return {"out": molt.moe_layer(s["x"], w["w_router"], w["w_gate_up"], w["w_down"], BIG["K"],
                                      router_bias=w["router_bias"], s_gate_up=w["s_gate_up"],
                                      s_down=w["s_down"], workspace=s["ws"], packed=True)}
    caches = {"k_cache": s["kc"], "v_cache": s["vc"]}
    if kind == "layer":
        x = s["x"].clone()      # the layer updates the residual stream in place
        molt.decoder_forward(s["model"], s["kv"], case["B"], case["k"], x, workspace=s["ws"])
        return dict(caches, x=x)
    if kind == "prefill":
        out = molt.prefill(s["model"], s["kv"], s["tokens"], s["lens"], want_hidden=True, workspace=s["ws"])
    else:
        out = molt.score_tokens(s["model"], s["kv"], s["tokens"], s["targets"], replay_routes=s["routes"],
                                want_logits=True, workspace=s["ws"])
    return dict(caches, **out)


# ---------------------------------------------------------------------------- work

def _touched(case, T, E, K):
    """Expected number of experts that T rows reach."""
    z = case.get("zipf", 0.0) or 0.0
    p = [(r + 1) ** -z for r in range(E)]
    t = sum(p)
    return sum(1.0 - (1.0 - min(1.0, K * v / t)) ** T for v in p)


def _moe_work(case, m, T):
    d, E, K, F = m["d"], m["E"], m["K"], m["F"]
    es = {"f32": 4, "bf16": 2, "fp8": 1}[case["experts"]]
    es_r = 4 if case["experts"] == "f32" else 2
    return _touched(case, T, E, K) * 3 * d * F * es + E * d * es_r, 6.0 * T * K * d * F + 2.0 * T * d * E


def work(case):
    if case["kind"] == "accept":
        B, k, V = case["B"], case["k"], case["V"]
        rows = B * (k + 1) + B * (1 if case["q"] and k else 0)      # every logit, one q row a sequence
        return {"bytes": 4.0 * rows * V, "flops": 2.0 * B * (k + 1) * V}
    if case["kind"] == "moe":
        b, f = _moe_work(case, BIG, case["T"])
        return {"bytes": b + case["T"] * BIG["d"] * (2 + 4), "flops": f}
    m, B = _dims(case), case["B"]
    n = case["n"] if case["kind"] == "prefill" else case["k"] + 1
    L = 1 if case["kind"] == "layer" else 2
    T, c = B * n, 0.5 * (case["ctx_lo"] + case["ctx_hi"])
    d, D, es = m["d"], m["D"], 4 if case["experts"] == "f32" else 2
    proj = (m["Hq"] + 2 * m["Hkv"]) * D * d + m["Hq"] * D * d
    mb, mf = _moe_work(case, m, T)
    kv = B * (c + n) * m["Hkv"] * D * 2 * es            # cached keys and values read, new ones written
    nbytes = L * (mb + proj * es + kv) + 2 * T * d * 4
    flops = L * (mf + 2.0 * T * proj + 4.0 * m["Hq"] * D * T * (c + 0.5 * (n + 1)))
    if case["kind"] != "layer":
        rows = B if case["kind"] == "prefill" else T
        nbytes += m["V"] * d * es + rows * m["V"] * 4
        flops += 2.0 * rows * m["V"] * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # bf16 storage of the norm outputs, q/k/v, the attention output and the SwiGLU product: a
    # sum in another order moves some of them by one bf16 step (2^-8), fp8 row codes by one fp8
    # step (2^-3). Measured against 64-bit sums with the same storage: layers 4e-5 to 1.7e-4,
    # with fp8 experts 1.3e-3; the expert block alone 5e-3 in fp8; logits after two layers
    # 1.1e-3; f32 3e-7; log-probs of the accept rule 2.7e-8 (f32 rounding). About four times
    # that; max covers one step of a single stored value and a few in one row.
    if case["kind"] == "accept":
        return {"rel": 2e-7, "max": 2e-6}        # whole values the same
    if case["experts"] == "f32":
        return {"rel": 2e-6, "max": 1e-4}
    if case["kind"] == "moe":
        return {"rel": 2e-2, "max": 0.5} if case["experts"] == "fp8" else {"rel": 5e-3, "max": 0.2}
    if case["kind"] == "layer":
        return {"rel": 5e-3, "max": 0.2} if case["experts"] == "fp8" else {"rel": 1e-3, "max": 0.05}
    return {"rel": 5e-3, "max": 0.2}


# ---------------------------------------------------------------------------- 64-bit results

def _rope(v, pos, D):
    half = D // 2
    inv = THETA ** (-2.0 * torch.arange(half, device="cuda", dtype=torch.float64) / D)
    a = pos.double()[:, None, None] * inv
    lo, hi = v[..., :half], v[..., half:]
    return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)


def _norm(x, g):
    return x / (x.square().mean(-1, keepdim=True) + EPS).sqrt() * g.double()


def _codes(v):
    """The per-row fp8 quantisation of the format's definition: values and scales."""
    s = v.abs().amax(-1, keepdim=True).float() / 448.0
    q = (v.float() / s).nan_to_num(0.0).to(torch.float8_e4m3fn)
    return q.double(), s.double()


def _exact_moe(y, w, K, rnd, fp8, replay=None):
    """Expert sum of rows y (f64, already in the storage type)."""
    E, twoF, _ = w["w_gate_up"].shape
    F = twoF // 2
    g = y @ w["w_router"].double().T
    if w["router_bias"] is not None:
        g = g + w["router_bias"].double()
    ids = g.topk(K, -1).indices if replay is None else replay.long()
    p = torch.softmax(g.gather(1, ids), -1)
    rows, sc = _codes(y) if fp8 else (y, 1.0)
    out = torch.zeros_like(y)
    for e in range(E):
        t, j = (ids == e).nonzero(as_tuple=True)
        if t.numel() == 0:
            continue
        gu, dn = w["w_gate_up"][e], w["w_down"][e]
        if fp8:
            gu = gu.view(torch.float8_e4m3fn).double() * w["s_gate_up"][e].double()[:, None]
            dn = dn.view(torch.float8_e4m3fn).double() * w["s_down"][e].double()[:, None]
        v = (rows[t] @ gu.double().T) * (sc[t] if fp8 else 1.0)
        h = rnd(v[:, :F] * torch.sigmoid(v[:, :F]) * v[:, F:])
        if fp8:
            hq, hs = _codes(h)
            h = hq * hs
        out.index_add_(0, t, (h @ dn.double().T) * p[t, j][:, None])
    return out


def _exact_layer(case, s, l, x, rnd):
    m, kp1 = _dims(case), s["kp1"]
    B, Hq, Hkv, D = case["B"], m["Hq"], m["Hkv"], m["D"]
    w, T = s["layers"][l], case["B"] * kp1
    pos = (s["ctx"].long()[:, None] + torch.arange(kp1, device="cuda")).reshape(-1)
    qkv = (rnd(_norm(x, w["attn_norm"])) @ w["w_qkv"].double().T).view(T, Hq + 2 * Hkv, D)
    qk = rnd(_rope(qkv[:, :Hq + Hkv], pos, D)).view(B, kp1, Hq + Hkv, D)
    v = rnd(qkv[:, Hq + Hkv:]).view(B, kp1, Hkv, D)
    att = torch.empty(B, kp1, Hq, D, dtype=torch.float64, device="cuda")
    for b in range(B):
        c = int(s["ctx"][b])
        blocks = s["bt"][b, :(c + 15) // 16].long()
        keys = s["kc"][l][blocks].permute(1, 0, 2, 3).reshape(Hkv, -1, D)[:, :c].double()
        vals = s["vc"][l][blocks].permute(1, 0, 3, 2).reshape(Hkv, -1, D)[:, :c].double()
        keys = torch.cat([keys, qk[b, :, Hq:].transpose(0, 1)], 1)
        vals = torch.cat([vals, v[b].transpose(0, 1)], 1)
        hidden = torch.arange(c + kp1, device="cuda")[None, :] > c + torch.arange(kp1, device="cuda")[:, None]
        for h in range(Hkv):
            q = qk[b, :, h * (Hq // Hkv):(h + 1) * (Hq // Hkv)].transpose(0, 1)     # [G, kp1, D]
            sc = (q @ keys[h].T / math.sqrt(D)).masked_fill_(hidden, -math.inf)
            att[b, :, h * (Hq // Hkv):(h + 1) * (Hq // Hkv)] = (torch.softmax(sc, -1) @ vals[h]).transpose(0, 1)
    x = x + rnd(att.view(T, Hq * D)) @ w["w_o"].double().T
    y = rnd(_norm(x, w["moe_norm"]))
    replay = s["routes"][l] if "routes" in s else None
    return x + _exact_moe(y, w, m["K"], rnd, case["experts"] == "fp8", replay)


def _exact_accept(case, seed):
    s = _accept_inputs(case, seed)
    B, k, V = case["B"], case["k"], case["V"]
    z = s["logits"].double()
    lp = z - torch.logsumexp(z, -1, keepdim=True)
    p, u = lp.exp(), s["u"].double()
    tokens = torch.full((B, k + 1), -1, dtype=torch.int64, device="cuda")
    out = torch.full((B, k + 1), math.nan, dtype=torch.float64, device="cuda")
    n = torch.zeros(B, dtype=torch.int64, device="cuda")
    alive = torch.ones(B, dtype=torch.bool, device="cuda")
    at = torch.arange(B, device="cuda")
    for i in range(k):
        x = s["drafts"][:, i].long()
        q = s["q"][at, i, x].double() if s["q"] is not None else 1.0
        alive &= u[:, i] * q < p[at, i, x]
        tokens[alive, i], out[alive, i] = x[alive], lp[at, i, x][alive]
        n += alive
    r = p[at, n].clone()
    short = n < k
    if k > 0:
        j = n.clamp(max=k - 1)
        if s["q"] is not None:
            less = s["q"][at, j].double()
        else:
            less = torch.zeros_like(r).scatter_(1, s["drafts"].long()[at, j][:, None], 1.0)
        r = torch.where(short[:, None], (r - less).clamp_(min=0.0), r)
    r = torch.where(r.sum(-1, keepdim=True) > 0, r, p[at, n])
    cdf = (r * 2.0 ** 62).long().cumsum(-1)
    u32, tot = (u[:, k] * 2.0 ** 32).long(), cdf[:, -1]
    target = (tot >> 32) * u32 + (((tot & 0xFFFFFFFF) * (u32 >> 1)) >> 31)
    t = (cdf <= target[:, None]).sum(-1).clamp(max=V - 1)
    tokens[at, n], out[at, n] = t, lp[at, n, t]
    return {"tokens": tokens.int(), "n_accepted": n.int(), "logprobs": out}


def exact(case, seed):
    """run()'s result in 64 bits, with the storage types the entry points document (bf16 norm
    outputs, q/k/v, attention output and SwiGLU product; fp8 row codes). The caches have no
    such value: they are stored in 16 bits."""
    if case["kind"] == "accept":
        return _exact_accept(case, seed)

    def rnd(v):
        return v if case["experts"] == "f32" else v.to(BF16).double()

    if case["kind"] == "moe":
        s = _moe_inputs(case, seed)
        return {"out": _exact_moe(s["x"].double(), s["w"], BIG["K"], rnd, case["experts"] == "fp8")}
    s = _inputs(case, seed)
    L = len(s["layers"])
    caches = {"k_cache": [None] * L, "v_cache": [None] * L}
    if case["kind"] == "layer":
        return dict(caches, x=_exact_layer(case, s, 0, s["x"].double(), rnd))
    x = s["head"]["embed"][s["tokens"].long().reshape(-1)].double()
    for l in range(L):
        x = _exact_layer(case, s, l, x, rnd)
    rows = x
    if case["kind"] == "prefill":
        rows = x.view(case["B"], s["kp1"], -1)[torch.arange(case["B"], device="cuda"), s["lens"].long() - 1]
    logits = rnd(_norm(rows, s["head"]["final_norm"])) @ s["head"]["lm_head"].double().T
    if case["kind"] == "prefill":
        return dict(caches, logits=logits, hidden=x)
    logits = logits.view(case["B"], s["kp1"], -1)
    lp = logits - torch.logsumexp(logits, -1, keepdim=True)
    return dict(caches, logits=logits, logprobs=lp.gather(2, s["targets"].long()[..., None])[..., 0])
