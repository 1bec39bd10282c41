"""What the performance of this framework is measured on: passes through its public entry points
(s2o_plan, s2o_plan_static, s2o_attention, s2o_attention_local, s2o_attention_prefix) over the
shapes, thresholds and options of its own workloads, tests and studies.

A case is a dict of plain values:
  kind      layer   one attention layer of a prefill as bench.py enqueues it: the own-segment pass on
                    a second stream beside the ranking, then the prefix walk; all buffers kept
            calls   the plainest use: s2o_plan and s2o_attention one after the other, outputs and
                    scratch allocated by the calls
            fused   s2o_plan, then s2o_attention in its single-launch form without a state buffer
            plan    the ranking alone; `scores`: with the score outputs; `static`: s2o_plan_static
            walk    the attention alone on maps that are already there (a further threshold or a
                    tile budget on the same ranking; non-causal as well)
            dense   attention over all keys in storage order without any map (non-causal)
  Z H Hkv L S BM    batch, query heads, key/value heads, tokens, segment length, query tile rows
  tau stop_mode budget q_perm non_causal    the options of s2o_params and the threshold
  layout    packed ([Z, heads, L, D]) or token ([Z, L, heads, D], described by strides)
  data      planted / bursts / mixed / noise: structure of the keys (see _make_qkv)
  visited   prefix tiles a query tile visits on average, counted once on these inputs (0: estimated)
"""
import math

import torch

import paper_2602_22575_amd as s2o

D = 128
DEV = "cuda:0"

_BASE = dict(kind="layer", Z=1, H=32, Hkv=8, L=8192, S=1024, BM=64, tau=1e-3, stop_mode=0, budget=0,
             q_perm=1, non_causal=0, layout="packed", data="planted", scores=0, static=0,
             visited=0.0)


def _case(name, **kw):
    return dict(_BASE, name=name, **kw)


def listed():
    return [
        # the smallest complete use: one head, 2K tokens; latency and launches are all of it
        _case("tiny_2k", kind="calls", H=1, Hkv=1, L=2048, S=256, tau=0.05, visited=4.1),
        # a model that keeps its tensors token-major, a batch of two, a segment length that is no
        # power of two and an odd number of segments
        _case("ragged_token_major", kind="calls", Z=2, H=12, Hkv=4, L=7360, S=320, tau=5e-3, layout="token", visited=20.4),
        # one layer of the Llama-3.1-8B head shape at growing context, at the thresholds the
        # workloads are run with
        _case("llama_8k", L=8192, S=1024, tau=1e-3, visited=30.0),
        _case("llama_32k_bursts", L=32768, S=2048, tau=1e-3, data="bursts", visited=83.0),
        _case("llama_128k", L=131072, S=2048, tau=5e-3, visited=29.0),
        # half of the heads without structure (the stop rule rarely fires), 128-row query tiles
        _case("mixed_128k_bm128", L=131072, S=2048, tau=5e-3, BM=128, data="mixed", visited=150.0),
        # skipping switched off: must equal dense causal attention, all of the work is done
        _case("llama_32k_no_skipping", L=32768, S=2048, tau=0.0),
        # the ranking alone: with its scores and short segments (many rows), and on the built-in
        # scratch for callers that cannot allocate
        _case("plan_scores_64k", kind="plan", L=65536, S=1024, scores=1),
        _case("plan_static_4k", kind="plan", L=4096, S=512, static=1),
        # no memory for the state buffer: everything of the attention in one launch, queries in
        # original order (the paper's Alg. 4)
        _case("fused_16k_original_order", kind="fused", L=16384, S=1024, tau=5e-3, q_perm=0, visited=22.2),
        # a fixed budget of ranked key tiles instead of the stop rule, without causality, on maps
        # that are kept (top-k selection)
        _case("topk_16k_non_causal", kind="walk", H=16, Hkv=4, L=16384, S=2048, stop_mode=2, budget=64, tau=0.0,
              non_causal=1),
        # contiguous attention over all keys, no map (the baseline of the overhead study)
        _case("dense_8k_non_causal", kind="dense", L=8192, S=8192, stop_mode=2, tau=0.0, non_causal=1, q_perm=0,
              data="noise"),
    ]


def _work_units(c):
    """Rough cost in query-tile x key-tile products plus ranked keys, to keep drawn cases small."""
    w = work(c)
    return w["flops"] / 1e12 + w["bytes"] / 4e9


def draw(rng):
    most = 0.8 * max(_work_units(c) for c in listed())
    while True:
        c = dict(_BASE)
        c["kind"] = rng.choice(["layer", "layer", "layer", "calls", "calls", "fused", "plan", "plan", "walk", "dense"])
        c["H"], c["Hkv"] = rng.choice([(1, 1), (2, 1), (4, 2), (8, 8), (12, 4), (16, 4), (32, 8), (32, 8)])
        c["Z"] = rng.choice([1, 1, 1, 2, 3])
        c["BM"] = rng.choice([64, 64, 128])
        # segment length and number of segments over the logarithm of their ranges
        step = c["BM"]
        c["S"] = step * max(1, int(round(2 ** rng.uniform(0, 6) * 64 / step)))
        n = int(round(2 ** rng.uniform(1, 6)))
        if c["kind"] == "dense":
            n, c["non_causal"], c["q_perm"], c["stop_mode"], c["tau"], c["data"] = 1, 1, 0, 2, 0.0, "noise"
            c["S"] = step * rng.randint(512 // step, 8192 // step)
        c["L"] = n * c["S"]
        if c["L"] < 512 or c["L"] > 131072:
            continue
        if c["kind"] == "plan":
            c["scores"] = rng.choice([0, 1])
        if c["kind"] in ("layer", "calls", "fused", "walk"):
            c["tau"] = rng.choice([0.0, 10 ** rng.uniform(-4, -1.3), 10 ** rng.uniform(-3, -1.3)])
            c["stop_mode"] = rng.choice([0, 0, 0, 1])
            c["q_perm"] = rng.choice([1, 1, 0])
            c["layout"] = rng.choice(["packed", "packed", "token"])
            c["data"] = rng.choice(["planted", "planted", "bursts", "mixed", "noise"])
        if c["kind"] == "walk":
            c["non_causal"] = rng.choice([0, 1])
            if rng.random() < 0.5:
                c["stop_mode"], c["budget"] = 2, rng.randint(1, max(1, c["L"] // 128))
        if c["non_causal"] and c["L"] > 32768:      # rows of L ranked keys for every segment
            continue
        if c["Z"] * c["H"] * c["L"] > 32 * 131072 or _work_units(c) > most:
            continue
        return c


# ---------------------------------------------------------------------------------- inputs
def _ar1(noise, rho):
    """w_t = rho * w_{t-1} + noise_t along dim 0 of [L, D], in blocks: within a block by a
    triangular matrix of powers, between blocks by a second one."""
    L = noise.shape[0]
    b = 256
    n = (L + b - 1) // b
    x = torch.zeros((n * b, noise.shape[1]), dtype=torch.float32, device=noise.device)
    x[:L] = noise
    x = x.view(n, b, -1)

    def powers(k, r):
        e = torch.arange(k, device=noise.device)
        e = (e[:, None] - e[None, :]).to(torch.float64)
        return torch.where(e >= 0, torch.exp(e.clamp(min=0) * math.log(r)), torch.zeros_like(e)).to(torch.float32)

    inside = torch.matmul(powers(b, rho), x)
    ends = torch.matmul(powers(n, rho ** b), inside[:, -1])            # true value at the end of every block
    carry = torch.zeros_like(ends)
    carry[1:] = ends[:-1]
    decay = torch.exp(torch.arange(1, b + 1, device=noise.device, dtype=torch.float64) * math.log(rho)).to(torch.float32)
    return (inside + decay[None, :, None] * carry[:, None, :]).reshape(n * b, -1)[:L]


def _make_qkv(c, seed):
    """The structure of the workloads in paper_2602_22575_amd/inputs.py, drawn on the GPU: N(0,1)
    plus, per key/value head, a direction u added to every query and (boosted) to the sinks and a
    few heavy keys, and a slow positional component shared by queries and keys."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    Z, H, Hkv, L = c["Z"], c["H"], c["Hkv"], c["L"]
    G = H // Hkv

    def randn(*shape):
        return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32)

    Q = torch.empty((Z, H, L, D), dtype=torch.bfloat16, device=DEV)
    K = torch.empty((Z, Hkv, L, D), dtype=torch.bfloat16, device=DEV)
    V = torch.empty((Z, Hkv, L, D), dtype=torch.bfloat16, device=DEV)
    for z in range(Z):
        for g in range(Hkv):
            k = randn(L, D)
            V[z, g] = randn(L, D)
            planted = c["data"] in ("planted", "bursts") or (c["data"] == "mixed" and g >= Hkv // 2)
            shared = None
            if planted:
                u = randn(D)
                u /= u.norm()
                strength = 0.2 + 0.6 * torch.rand((1,), generator=gen, device=DEV)
                shared = _ar1(0.05 * randn(L, D), 1.0 - 1.0 / 4096.0) * strength
                k += shared
                heavy = torch.zeros(L, dtype=torch.bool, device=DEV)
                heavy[:4] = True
                if c["data"] == "bursts":
                    at = torch.randint(0, max(1, L - 32), (16,), generator=gen, device=DEV)
                    heavy[(at[:, None] + torch.arange(32, device=DEV)[None, :]).clamp(max=L - 1).reshape(-1)] = True
                else:
                    heavy |= torch.rand((L,), generator=gen, device=DEV) < (0.01 if L <= 2048 else 0.005)
                k += heavy[:, None] * ((5.0 if c["data"] == "mixed" else 3.0) * u)[None, :]
            K[z, g] = k
            for j in range(G):
                q = randn(L, D)
                if planted:
                    q += shared
                    q += u
                Q[z, g * G + j] = q
    return Q, K, V


def _token_major(x):
    """[Z, heads, L, D] -> the same values stored as [Z, L, heads, D]."""
    return x.permute(0, 2, 1, 3).contiguous()


def prepare(case, seed):
    c = dict(case)
    Q, K, V = _make_qkv(c, seed)
    strides = {}
    if c["layout"] == "token":
        Q, K, V = (_token_major(x) for x in (Q, K, V))
        qs, ks = (c["L"] * c["H"] * D, D, c["H"] * D), (c["L"] * c["Hkv"] * D, D, c["Hkv"] * D)
        strides = dict(q_stride=qs, k_stride=ks, v_stride=ks, o_stride=qs)
    p = s2o.make_params(c["Z"], c["H"], c["Hkv"], c["L"], D, c["S"], c["BM"], 64, use_q_perm=c["q_perm"],
                        stop_mode=c["stop_mode"], max_prefix_tiles=c["budget"], non_causal=c["non_causal"], **strides)
    s = {"c": c, "p": p, "Q": Q, "K": K, "V": V}
    Z, H, L, S = c["Z"], c["H"], c["L"], c["S"]
    N = L // S
    if c["layout"] == "token":                       # the output buffer of such a model is token-major too
        s["O"] = torch.empty_like(Q)
    if c["kind"] == "layer":
        P = S * N * (N - 1) // 2
        s["maps"] = (torch.empty((Z, H, N, S), dtype=torch.int32, device=DEV),
                     torch.empty((Z, H, max(P, 4)), dtype=torch.int32, device=DEV))
        s["plan_scratch"] = torch.empty(s2o.s2o_plan_sizes(p)["scratch"], dtype=torch.uint8, device=DEV)
        s["state"] = torch.empty(s2o.s2o_attention_sizes(p)["scratch"], dtype=torch.uint8, device=DEV)
        s.setdefault("O", torch.empty((Z, H, L, D), dtype=torch.bfloat16, device=DEV))
        s["counts"] = tuple(torch.empty((Z, H, L // c["BM"]), dtype=torch.int32, device=DEV) for _ in range(2))
        s["side"] = torch.cuda.Stream()
    elif c["kind"] == "walk":
        plan = s2o.s2o_plan(Q, K, p, want_scores=False)
        s["maps"] = (plan.q_perm, plan.kv_perm)
        if not c["non_causal"]:
            s["state"] = s2o.s2o_attention_local(Q, K, V, p)
        torch.cuda.synchronize()
    return s


# ------------------------------------------------------------------------------------ pass
def run(s):
    c, p, Q, K, V = s["c"], s["p"], s["Q"], s["K"], s["V"]
    if c["kind"] == "layer":
        main, side = torch.cuda.current_stream(), s["side"]
        fork = torch.cuda.Event()
        fork.record(main)
        side.wait_event(fork)
        s2o.s2o_attention_local(Q, K, V, p, scratch=s["state"], stream=side)
        join = torch.cuda.Event()
        join.record(side)
        plan = s2o.s2o_plan(Q, K, p, want_scores=False, scratch=s["plan_scratch"], maps=s["maps"])
        main.wait_event(join)
        out = s2o.s2o_attention_prefix(Q, K, V, p, plan.q_perm, plan.kv_perm, c["tau"], s["state"], O=s["O"],
                                       computed=s["counts"][0], skipped=s["counts"][1])
        return [plan.q_perm, plan.kv_perm, *out]
    if c["kind"] == "plan":
        plan = s2o.s2o_plan(Q, K, p, want_scores=bool(c["scores"]), static_scratch=bool(c["static"]))
        return [plan.q_perm, plan.kv_perm, plan.s_q, plan.s_k, plan.q_mean, plan.k_guide]
    if c["kind"] in ("calls", "fused"):
        plan = s2o.s2o_plan(Q, K, p, want_scores=False)
        out = s2o.s2o_attention(Q, K, V, p, plan.q_perm, plan.kv_perm, c["tau"], O=s.get("O"),
                                two_pass=c["kind"] == "calls")
        return [plan.q_perm, plan.kv_perm, *out]
    if c["kind"] == "walk":
        return list(s2o.s2o_attention_prefix(Q, K, V, p, *s["maps"], c["tau"], s.get("state"), O=s.get("O")))
    return list(s2o.s2o_attention(Q, K, V, p, None, None, c["tau"]))


# ---------------------------------------------------------------------------- work, tolerance
def _prefix_tiles(c):
    """Nominal number of 64-token prefix tiles all query tiles of one head visit.  The stop rule
    makes it depend on the data: 0.66 * tau^-0.78 tiles per query tile is what the planted
    inputs show at 128K (145 at 1e-3, 41 at 5e-3, 15 at 2e-2); heads without structure walk about
    5.5 times as far."""
    N, nq = c["L"] // c["S"], c["S"] // c["BM"]
    if c["visited"]:
        return c["visited"] * N * nq
    far = {"noise": 5.5, "mixed": 3.25}.get(c["data"], 1.0)
    total = 0.0
    for n in range(N):
        k = (c["L"] if c["non_causal"] else n * c["S"]) // 64
        if c["budget"]:
            k = min(k, c["budget"])
        if c["stop_mode"] != 2 and c["tau"] > 0:
            k = min(k, far * 0.66 * c["tau"] ** -0.78)
        total += k * nq
    return total


def work(case):
    """bytes: inputs and outputs of the pass once each; flops: QK^T and PV on the own-segment
    triangle and the visited prefix tiles, and the ranking's one dot product per query and per
    (segment, prefix key)."""
    c = case
    Z, H, Hkv, L, S = c["Z"], c["H"], c["Hkv"], c["L"], c["S"]
    N = L // S
    P = N * L if c["non_causal"] else S * N * (N - 1) // 2
    q, kv = Z * H * L * D * 2, Z * Hkv * L * D * 2
    maps = Z * H * (L + P) * 4
    plan_flops = Z * H * 2.0 * D * (L + P)
    if c["kind"] == "plan":
        scores = (Z * H * (L + P + N * D) * 4 + Z * Hkv * D * 4) if c["scores"] else 0
        return {"bytes": q + kv + maps + scores, "flops": plan_flops}
    visited = _prefix_tiles(c)
    flops = 4.0 * c["BM"] * 64 * D * visited * Z * H
    counts = 2 * Z * H * (L // c["BM"]) * 4
    attn_bytes = 2 * q + 2 * kv + counts
    if c["kind"] == "dense":
        return {"bytes": attn_bytes, "flops": flops}
    if not c["non_causal"] and c["kind"] != "walk":
        flops += Z * H * N * 4.0 * D * (S * (S + 1) / 2)
    if c["kind"] == "walk":                          # the maps are read, the ranked rows as far as they are walked
        state = 0 if c["non_causal"] else Z * H * L * (D + 2) * 4
        rows = min(P, visited / max(1, S // c["BM"]) * 64)
        return {"bytes": attn_bytes + state + Z * H * (L + rows) * 4, "flops": flops}
    return {"bytes": attn_bytes + maps, "flops": flops + plan_flops}


def tolerance(case):
    """Measured against the same path with its sums in another order (own-segment tiles in the
    fused launch's order: O off by 1.4e-5 in the 2-norm and by one bf16 ulp, 1.2e-2, at most) and
    against 64-bit scores (scores off by 6e-8 in the 2-norm, 3.5e-7 at most; 7e-4 of the map
    entries of 64K tokens differ, all near-ties).  For O the limit is that of bf16 results with
    bf16 softmax numerators formed against another reference maximum (2^-9 each); a stop decision
    that falls the other way on a near-tie moves a few rows by about the threshold."""
    if case["kind"] == "plan":
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}
    return {"rel": 5e-3, "max": 0.2, "differ": 1e-3}
