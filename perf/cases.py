"""The work that a user of this framework has it do, as cases that can be timed and compared.

A case is one pass over one batch through the public entry points: a reversible training step (forward, then the sweep
step that rebuilds the input and takes all gradients), the same as three separate calls, the stored-activation
comparison, a stack of blocks, or the passes without gradients on pre-merged adapter weights.  Geometries are those of
the repository's workloads, benchmark and parity tests; batch and sequence lengths run from one token to the longest
sequence of the benchmark, ragged ones among them.
"""
import math

import torch

import paper_2512_20920_amd as R
from paper_2512_20920_amd import harness

# d_model, heads, head width, experts, top-k, expert width, shared-expert width
QWEN = dict(d_model=2048, n_heads=16, head_dim=128, n_experts=60, top_k=4, d_expert=1408, d_shared=5632)
FEWBIG = dict(d_model=4096, n_heads=32, head_dim=128, n_experts=8, top_k=2, d_expert=14336, d_shared=0)
MID = dict(d_model=512, n_heads=4, head_dim=128, n_experts=12, top_k=3, d_expert=192, d_shared=320)
NARROW = dict(d_model=256, n_heads=4, head_dim=64, n_experts=15, top_k=4, d_expert=360, d_shared=448)
TINY = dict(d_model=64, n_heads=4, head_dim=16, n_experts=8, top_k=2, d_expert=128, d_shared=0)

# op: "step" = forward + inverse_backward, "calls" = forward + inverse + backward, "stored" = forward + backward_stored,
#     "stack" = stack_forward + stack_backward over `blocks` blocks, "merged" = forward_merged + inverse_merged
# train: which weight gradients are asked for ("all"; "stage1" = the four adapters; "stage2" = all but the router)
DEFAULTS = dict(op="step", dtype="bf16", blocks=1, train="all", iters=1, fp32_streams=False, fp32_grads=False, skewed=False)

ADAPTERS = ("pup_a", "pdn_a", "pup_m", "pdn_m")


def _case(name, geometry, B, S, **options):
    return dict(dict(DEFAULTS, name=name, **geometry), B=B, S=S, **options)


def listed():
    return [
        # the float32 block small enough for a reference in double precision: every launch counts
        _case("tiny_f32_calls", TINY, 2, 32, dtype="f32", op="calls"),
        # float32 twin of a mid-sized block: checking gradients or numerics against the bf16 run
        _case("mid_f32_step", MID, 2, 200, dtype="f32"),
        # a reduced bf16 block, ragged tails in every dimension: experiments on a small model
        _case("mid_bf16_step", MID, 2, 200),
        # the same kind of model with heads 64 wide
        _case("narrow_heads_step", NARROW, 3, 251),
        # a short prompt through static weights: forward, and the input rebuilt from the output
        _case("prompt_merged", QWEN, 1, 37, op="merged"),
        # one short example per step
        _case("qwen_b1s128_step", QWEN, 1, 128),
        # the headline training batch
        _case("qwen_b4s512_step", QWEN, 4, 512),
        # first training stage (adapters only), float32 residual streams, two fixed-point iterations, ragged batch
        _case("qwen_stage1_b3s333", QWEN, 3, 333, train="stage1", fp32_streams=True, iters=2),
        # imbalanced routing: a router bias gives the hottest expert about 8 times the mean
        _case("qwen_skewed_b2s2048", QWEN, 2, 2048, skewed=True),
        # long context, where attention weighs most
        _case("qwen_b1s8192_step", QWEN, 1, 8192),
        # forward through a stack that keeps the last state only, and the sweep back down
        _case("qwen_stack4_b1s1024", QWEN, 1, 1024, op="stack", blocks=4),
        # few large experts: the compute-bound end of the routed GEMMs
        _case("fewbig_b2s1024_step", FEWBIG, 2, 1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _batch(rng, lo, hi, most_s):
    """(B, S) with B * S spread over the logarithm of [lo, hi]."""
    T = _log_int(rng, lo, hi)
    B = min(T, max(rng.choice((1, 1, 2, 3, 4, 8)), -(-T // most_s)))
    return B, max(1, T // B)


def draw(rng):
    kind = rng.choice(("qwen",) * 6 + ("merged",) * 2 + ("mid",) * 3 + ("f32",) * 2 + ("stack", "fewbig"))
    opt = {}
    if kind == "qwen":
        B, S = _batch(rng, 16, 8192, 8192)
        geo = QWEN
        opt["op"] = rng.choice(("step", "step", "step", "calls", "stored"))
        if opt["op"] == "calls":
            B, S = _batch(rng, 16, 4096, 4096)
        opt["train"] = rng.choice(("all", "all", "stage1", "stage2"))
        opt["fp32_streams"] = rng.random() < 0.3
        opt["fp32_grads"] = rng.random() < 0.2
        opt["skewed"] = rng.random() < 0.25
        opt["iters"] = rng.choice((1, 1, 2)) if B * S <= 4096 else 1
    elif kind == "merged":
        B, S = _batch(rng, 1, 8192, 8192)
        geo, opt["op"], opt["fp32_streams"] = QWEN, "merged", rng.random() < 0.3
    elif kind == "mid":
        B, S = _batch(rng, 17, 2048, 1024)
        dh = rng.choice((64, 128))
        H = rng.randint(2, 1024 // dh)
        E = rng.randint(4, 24)
        geo = dict(d_model=H * dh, n_heads=H, head_dim=dh, n_experts=E, top_k=rng.randint(1, 4),
                   d_expert=8 * rng.randint(8, 90), d_shared=rng.choice((0, 8 * rng.randint(8, 180))))
        opt["op"] = rng.choice(("step", "calls", "stored", "merged"))
        opt["fp32_streams"] = rng.random() < 0.3
    elif kind == "f32":
        B, S = _batch(rng, 16, 1024, 512)
        H, dh = rng.randint(2, 8), rng.choice((16, 32, 64))
        E = rng.randint(4, 16)
        geo = dict(d_model=H * dh, n_heads=H, head_dim=dh, n_experts=E, top_k=rng.randint(1, 4),
                   d_expert=8 * rng.randint(6, 32), d_shared=rng.choice((0, 8 * rng.randint(6, 48))))
        opt["dtype"], opt["op"] = "f32", rng.choice(("step", "calls", "merged"))
    elif kind == "stack":
        B, S = _batch(rng, 64, 1024, 1024)
        geo, opt["op"], opt["blocks"], opt["fp32_streams"] = QWEN, "stack", rng.randint(2, 4), rng.random() < 0.3
    else:
        B, S = _batch(rng, 64, 2048, 2048)
        geo = FEWBIG
        opt["fp32_streams"] = rng.random() < 0.3
    case = _case("", geo, B, S, **opt)
    del case["name"]
    return case


def _shapes(c):
    d, E, I, Is = c["d_model"], c["n_experts"], c["d_expert"], c["d_shared"]
    h = d // 2
    s = {"norm_a1": (h,), "norm_a2": (h,), "norm_m": (h,), "pup_a": (d, h), "pdn_a": (h, d), "pup_m": (d, h),
         "pdn_m": (h, d), "wq": (d, d), "wk": (d, d), "wv": (d, d), "wo": (d, d), "bq": (d,), "bk": (d,), "bv": (d,),
         "w_router": (E, d), "w_gate_up": (E, 2 * I, d), "w_down": (E, d, I)}
    if c["skewed"]:
        s["b_router"] = (E,)
    if Is:
        s.update(ws_gate_up=(2 * Is, d), ws_down=(d, Is), ws_gate=(d,))
    return s


def _wanted(c):
    skip = {"stage1": [n for n in R.WEIGHT_FIELDS if n not in ADAPTERS], "stage2": ["w_router", "b_router"]}
    return [n for n in _shapes(c) if n not in skip.get(c["train"], ())]


def _tokens_and_routers(c, W, gen):
    """Stream 1 of the batch, and routers that tell its tokens apart as trained ones do: every token is one of a few
    dozen kinds plus as much again of its own, and each block's router gives the kind's top-k experts logits of 3.5 and
    up against 0 for the rest.  (Random router weights leave a per cent of the tokens with two experts level to within
    the rounding of stream 1, and whole rows of the expert gradients then depend on which of the two is taken.)
    Skewed: experts are drawn by rank ** -0.8, which gives the hottest about 8 times the mean load at the Qwen shape."""
    E, k, h, dev = c["n_experts"], c["top_k"], c["d_model"] // 2, gen.device
    kinds = max(1, min(2 * E, h // 4))
    center = torch.randn((kinds, h), device=dev, generator=gen)
    for l in range(c["blocks"]):
        if c["skewed"]:
            rank = torch.randperm(E, device=dev, generator=gen) + 1.0
            chosen = torch.multinomial((rank ** -0.8).expand(kinds, -1), k, generator=gen)
        else:                             # every expert equally often
            rounds = [torch.randperm(E, device=dev, generator=gen) for _ in range(-(-kinds // E))]
            first = torch.cat(rounds)[:kinds]
            steps = torch.cat([torch.zeros(1, device=dev), 1 + torch.randperm(E - 1, device=dev, generator=gen)[:k - 1]])
            chosen = (first[:, None] + steps[None].long()) % E
        want = torch.zeros((kinds, E), device=dev)
        want.scatter_(1, chosen, 3.0 + 0.5 * torch.arange(k, 0, -1, device=dev).float().expand(kinds, -1))
        lifted = (center * center.square().mean(1, keepdim=True).rsqrt() * W["norm_m"][l].float()) @ W["pup_m"][l].float().T
        gram = (lifted @ lifted.T).double().cpu()
        W["w_router"][l] = want.T @ torch.linalg.solve(gram, lifted.double().cpu()).float().to(dev)
    kind = torch.randint(kinds, (c["B"] * c["S"],), device=dev, generator=gen)
    own = torch.randn((c["B"] * c["S"], h), device=dev, generator=gen)
    return (center[kind] + own) * 0.5 ** 0.5


def prepare(case, seed):
    c = case
    dev, L, h, T = "cuda", c["blocks"], c["d_model"] // 2, c["B"] * c["S"]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    sdt = torch.float32 if c["fp32_streams"] else dt
    gdt = torch.float32 if c["fp32_grads"] else dt
    gen = torch.Generator(dev).manual_seed(seed)

    def normal(shape, std, dtype, mean=0.0):
        return torch.empty(shape, dtype=dtype, device=dev).normal_(mean, std, generator=gen)

    # one tensor per weight over all blocks of a stack; the repository's recipe: N(0, 0.02), gains around 1
    W = {}
    for n, shape in _shapes(c).items():
        if n == "b_router":
            W[n] = normal((L,) + shape, 0.1, torch.float32)
        else:
            W[n] = normal((L,) + shape, 0.02, dt, 1.0 if n.startswith("norm_") else 0.0)
    x1 = _tokens_and_routers(c, W, gen)
    G = {n: torch.zeros_like(W[n], dtype=torch.float32 if n == "b_router" else gdt) for n in _wanted(c)}
    cfg = R.Config(**{k: c[k] for k in QWEN}, dtype=int(c["dtype"] == "bf16"), causal=1, use_rope=1, norm_topk_prob=0,
                   n_inv_iters=c["iters"], rope_theta=1.0e6, rms_eps=1.0e-6, fp32_streams=int(c["fp32_streams"]),
                   symmetric=0, fp32_grads=int(c["fp32_grads"]))
    s = dict(case=c, ctx=R.Context(cfg, c["B"], c["S"]), W=W, G=G)
    s["w"] = [R.binding._struct(R.Weights, {n: t[l] for n, t in W.items()}) for l in range(L)]
    s["g"] = [R.binding._struct(R.Grads, {n: t[l] for n, t in G.items()}) for l in range(L)]
    s["x1"], s["x2"] = x1.to(sdt), normal((T, h), 1.0, sdt)
    for n in ("dy1", "dy2"):
        s[n] = normal((T, h), 1.0, dt)
    for n in ("y1", "y2", "r1", "r2"):
        s[n] = torch.empty((T, h), dtype=sdt, device=dev)
    for n in ("dx1", "dx2"):
        s[n] = torch.empty((T, h), dtype=dt, device=dev)
    if c["op"] == "merged":
        class wl:
            d_model, n_experts, d_expert, d_shared, dtype = (c[k] for k in ("d_model", "n_experts", "d_expert", "d_shared", "dtype"))
        s["M"] = harness.alloc_merged(wl)
        s["m"] = R.binding._m(s["M"])
        R.revffn_merge_adapters(s["ctx"], s["w"][0], s["m"])
    return s


def run(state):
    s, c = state, state["case"]
    ctx, w, g, B, S, ld = s["ctx"], s["w"], s["g"], c["B"], c["S"], c["d_model"] // 2
    x1, x2, y1, y2, r1, r2 = (s[n] for n in ("x1", "x2", "y1", "y2", "r1", "r2"))
    dy1, dy2, dx1, dx2 = (s[n] for n in ("dy1", "dy2", "dx1", "dx2"))
    if c["op"] == "merged":
        R.revffn_forward_merged(ctx, w[0], s["m"], x1, x2, y1, y2, B, S, ld)
        R.revffn_inverse_merged(ctx, w[0], s["m"], y1, y2, r1, r2, B, S, ld)
        return [y1, y2, r1, r2]
    if c["op"] == "stack":
        R.revffn_stack_forward(ctx, w, x1, x2, y1, y2, B, S, ld)
        r1.copy_(y1), r2.copy_(y2), dx1.copy_(dy1), dx2.copy_(dy2)     # the sweep works in place
        R.revffn_stack_backward(ctx, w, g, r1, r2, dx1, dx2, B, S, ld)
    else:
        R.revffn_forward(ctx, w[0], x1, x2, y1, y2, B, S, ld)
        if c["op"] == "step":
            R.revffn_inverse_backward(ctx, w[0], y1, y2, r1, r2, dy1, dy2, dx1, dx2, g[0], B, S, ld)
        elif c["op"] == "calls":
            R.revffn_inverse(ctx, w[0], y1, y2, r1, r2, B, S, ld)
            R.revffn_backward(ctx, w[0], r1, r2, y1, dy1, dy2, dx1, dx2, g[0], B, S, ld)
        else:
            R.revffn_backward_stored(ctx, w[0], x1, x2, y1, dy1, dy2, dx1, dx2, g[0], B, S, ld)
            return [y1, y2, dx1, dx2, s["G"]]
    return [y1, y2, r1, r2, dx1, dx2, s["G"]]


def work(case):
    c = case
    d, E, k, I, Is, B, S, L = (c[n] for n in ("d_model", "n_experts", "top_k", "d_expert", "d_shared", "B", "S", "blocks"))
    h, T = d // 2, B * S
    es = 2 if c["dtype"] == "bf16" else 4
    ss, gs = (4 if c["fp32_streams"] else es), (4 if c["fp32_grads"] else es)
    hit = E * (1.0 - (1.0 - k / E) ** T)                      # experts that some token selects
    used = {n: math.prod(s) * (hit / E if n in ("w_gate_up", "w_down") else 1.0) for n, s in _shapes(c).items()}
    core = 2.0 * B * S * S * d                                # scores and values, half of them under the causal mask
    if c["op"] == "merged":
        q, kv, o = 2.0 * T * h * d, 4.0 * T * h * d, 2.0 * T * d * h
        moe = 2.0 * T * (3 * h * (k * I + Is) + E * h)
        half = {"wq", "wk", "wv", "wo", "w_gate_up", "w_down", "ws_gate_up", "ws_down"}
        weights = sum(v * 0.5 for n, v in used.items() if n in half) * es + (E + 1) * h * 4
        return {"bytes": weights + 6.0 * T * h * ss, "flops": 2.0 * moe + q * (1 + c["iters"]) + 2 * kv + (core + o) * (1 + c["iters"])}
    q, kv, o = 2.0 * T * d * (h + d), 2.0 * T * d * (h + 2 * d), 2.0 * T * d * (d + h)
    query = q + core + o                                      # the part of the attention half that an iterate repeats
    moe = 2.0 * T * (2 * d * h + 3 * d * (k * I + Is) + E * h)
    forward = query + kv + moe
    grads = 5.0 * B * S * S * d + q + kv + o + moe            # through the activations
    per_weight = {"pup_a": 2, "pup_m": 1, "pdn_a": 1, "pdn_m": 1, "wq": 1, "wk": 1, "wv": 1, "wo": 1, "w_router": 1,
                  "w_gate_up": k / E, "w_down": k / E, "ws_gate_up": 1, "ws_down": 1}
    shapes = _shapes(c)
    grads += sum(2.0 * T * math.prod(shapes[n]) * per_weight.get(n, 0) for n in _wanted(c))
    rebuild = {"step": kv + moe + query * (c["iters"] + 1), "stack": kv + moe + query * (c["iters"] + 1), "stored": 0.0,
               "calls": kv + moe + query * c["iters"] + forward}[c["op"]]
    weights = sum(v * (4 if n == "b_router" else es) for n, v in used.items())
    out = sum(math.prod(shapes[n]) * (4 if n == "b_router" else gs) for n in _wanted(c))
    streams = T * h * (ss * (6 if c["op"] != "stored" else 4) + es * 4)
    return {"bytes": L * (weights + out) + streams, "flops": L * (forward + rebuild + grads)}


def tolerance(case):
    if case["dtype"] == "f32":
        return {"rel": 2e-5}
    return {"rel": 2e-2}
