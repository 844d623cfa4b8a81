"""Performance cases of the rollout-allocation path.

Each case is one piece of work that a program using this package has it do,
through the package's public entry points, at the sizes of the package's own
workloads (the 1.5B- and 3B-shaped decoders and the tiny fp32 one) or generic
ones.  Layer-level cases keep a model's full width and cut its depth and, in
proportion, its vocabulary, so that the kernels run in about the mix that the
whole model has.

kind "sample"   the stand-alone sampler on given logits
kind "predict"  Eq. peff for a pool of prompts and Eq. grpo for its groups
kind "step"     a whole allocation step: prefill, decode / decide / refill to
                its end, advantages, read-back
kind "decode"   prefill of a prompt pool, then `steps` loop iterations from
                the captured graph and one more decode step that returns its
                logits (steps = 0: prefill and the first token)

Decode cases are teacher forced (random tokens, no EOS), so their logits are a
function of the inputs alone; a rollout's slot is its place in (prompt,
rollout) order.
"""
import math

import numpy as np
import torch

import paper_2607_26253_amd as sara

W_STD = 0.02          # random-init weights, as in the package's workloads
FORCED_EOS = (1 << 32) // 16


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def _model(layers, d, hq, hkv, hd, ffn, vocab, dtype="bf16"):
    return dict(layers=layers, d=d, hq=hq, hkv=hkv, hd=hd, ffn=ffn, vocab=vocab, dtype=dtype)


W15 = (1536, 12, 2, 128, 8960)      # width of the 1.5B-shaped decoder (28 layers, vocabulary 151936)
W3 = (2048, 16, 2, 128, 11008)      # width of the 3B-shaped decoder (36 layers)
TINY = (256, 4, 4, 64, 1024)        # the tiny fp32 decoder (2 layers, vocabulary 512)
FULL_V = 151936


def listed():
    return [
        # smallest calls: one interactive row through the sampler; the predictor and the
        # advantages of one step's pool
        dict(name="sample_one_row", kind="sample", rows=1, vocab=FULL_V, temperature=1.0, top_p=1.0, noalloc=True),
        dict(name="predict_and_score", kind="predict", prompts=256, groups=64, k=8),
        # nucleus sampling of a batch of rows from logits that the caller holds
        dict(name="sample_nucleus", kind="sample", rows=64, vocab=FULL_V, temperature=1.0, top_p=0.9, noalloc=True),
        # the tiny fp32 workload's whole step, as it is configured
        dict(name="step_tiny_f32", kind="step", **_model(2, *TINY, 512, "f32"), groups=16, k=8, n0=2, pool=64,
             slots=128, prompt_lo=32, prompt_hi=32, max_new=64, ragged=False),
        # a whole step of a small 64-wide-head decoder: odd prompt lengths, few slots (a queue), ragged rollouts
        dict(name="step_small_bf16", kind="step", **_model(2, 512, 8, 2, 64, 1408, 32016), groups=8, k=8, n0=2, pool=24,
             slots=24, prompt_lo=1, prompt_hi=77, max_new=24, ragged=True),
        # latency end of decode: one prompt's two probes
        dict(name="decode_two_rows", kind="decode", **_model(4, *W15, 32768), prompts=1, n0=2, slots=8, prompt_lo=200,
             prompt_hi=200, steps=128, top_p=1.0),
        # the benchmark's regime: the whole 1.5B-shaped model with about 32 of 512 slots occupied
        dict(name="decode_1p5b_32_rows", kind="decode", **_model(28, *W15, FULL_V), prompts=16, n0=2, slots=512,
             prompt_lo=128, prompt_hi=512, steps=64, top_p=1.0),
        # the start of a 1.5B step (64 prompts, two probes each) sampling from the nucleus
        dict(name="decode_nucleus_128_rows", kind="decode", **_model(2, *W15, FULL_V), prompts=64, n0=2, slots=512,
             prompt_lo=128, prompt_hi=512, steps=32, top_p=0.9),
        # full groups of the pool workload: 512 rows of the 3B width
        dict(name="decode_3b_512_rows", kind="decode", **_model(4, *W3, 32768), prompts=64, n0=8, slots=512,
             prompt_lo=256, prompt_hi=1024, steps=64, top_p=1.0),
        # contexts of thousands of tokens (the long-rollout workload's range)
        dict(name="decode_long_context", kind="decode", **_model(2, *W15, 32768), prompts=8, n0=4, slots=256,
             prompt_lo=3001, prompt_hi=4590, steps=128, top_p=1.0),
        # a step's prompt pool: prefill of 256 prompts to the first token of each
        dict(name="prefill_pool", kind="decode", **_model(4, *W15, 32768), prompts=256, n0=1, slots=512, prompt_lo=128,
             prompt_hi=512, steps=0, top_p=1.0),
        # few long prompts of the 3B width
        dict(name="prefill_long", kind="decode", **_model(4, *W3, 32768), prompts=3, n0=1, slots=64, prompt_lo=1100,
             prompt_hi=4590, steps=0, top_p=1.0),
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    widths = [W15, W15, W3, (512, 8, 2, 64, 1408), (1024, 16, 4, 64, 2816), (1024, 8, 1, 128, 4096)]
    while True:
        kind = rng.choice(["sample", "predict", "step", "decode", "decode", "decode", "prefill", "prefill"])
        if kind == "sample":
            top_p = rng.choice([1.0, 1.0, 0.95, 0.8, 0.3])
            return dict(kind="sample", rows=_log(rng, 1, 64 if top_p < 1.0 else 300),
                        vocab=rng.choice([_log(rng, 500, FULL_V), FULL_V]), temperature=rng.choice([1.0, 0.7, 1.3]),
                        top_p=top_p, noalloc=rng.random() < 0.7)
        if kind == "predict":
            return dict(kind="predict", prompts=_log(rng, 1, 4096), groups=_log(rng, 1, 512), k=rng.choice([2, 4, 8, 16, 31]))
        if kind == "step":
            f32 = rng.random() < 0.5
            w = rng.choice([TINY, (512, 8, 2, 64, 1408)]) if f32 else rng.choice(widths[3:])
            k = rng.choice([4, 8])
            groups, lo = _log(rng, 2, 16), rng.randint(1, 40)
            return dict(kind="step", **_model(rng.randint(1, 2), *w, 16 * rng.randint(32, 1024), "f32" if f32 else "bf16"),
                        groups=groups, k=k, n0=rng.choice([1, 2, 4]), pool=groups * rng.randint(2, 4),
                        slots=_log(rng, 8, 128), prompt_lo=lo, prompt_hi=lo + rng.randint(0, 60),
                        max_new=rng.randint(8, 40), ragged=rng.random() < 0.5)
        w = rng.choice(widths)
        vocab = 16 * rng.randint(256, 4096)
        lo = _log(rng, 16, 3000)
        hi = min(4590, _log(rng, lo, 4 * lo))
        if kind == "decode":
            prompts, n0 = _log(rng, 1, 64), rng.choice([1, 2, 2, 3, 4, 8])
            case = dict(kind="decode", **_model(rng.randint(1, 4), *w, vocab), prompts=prompts, n0=n0,
                        slots=max(prompts * n0, _log(rng, 8, 512)), prompt_lo=lo, prompt_hi=hi, steps=16 * rng.randint(1, 6),
                        top_p=rng.choice([1.0, 1.0, 1.0, 0.9]))
        else:
            prompts = _log(rng, 1, 256)
            case = dict(kind="decode", **_model(rng.randint(1, 4), *w, vocab), prompts=prompts, n0=1,
                        slots=max(prompts, _log(rng, 8, 512)), prompt_lo=lo, prompt_hi=hi, steps=0, top_p=1.0)
        if prompts * (lo + hi) / 2 <= 60000 and work(case)["flops"] <= 3e13:
            return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1000003 + stream) % (1 << 62))


def _weights(case, seed):
    """Device weights in sara_init's order (bf16 as tensors of torch.bfloat16)."""
    d, q, kv, f, V = case["d"], case["hq"] * case["hd"], case["hkv"] * case["hd"], case["ffn"], case["vocab"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = _gen(seed, 1)

    def mat(*shape):
        return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * W_STD).to(dt)

    def gain():
        return (1.0 + 0.1 * torch.randn(d, generator=g, device="cuda", dtype=torch.float32)).to(dt)

    out = [mat(V, d)]
    for _ in range(case["layers"]):
        out += [gain(), mat(q, d), mat(kv, d), mat(kv, d), mat(d, q), gain(), mat(f, d), mat(f, d), mat(d, f)]
    return out + [gain(), mat(V, d)]


def _descs(case):
    model = dict(n_layers=case["layers"], d_model=case["d"], n_heads=case["hq"], n_kv_heads=case["hkv"],
                 head_dim=case["hd"], d_ffn=case["ffn"], vocab=case["vocab"],
                 rope_theta=1.0e6 if case["dtype"] == "bf16" else 1.0e4, rms_eps=1e-6, dtype=case["dtype"],
                 eos_id=case["vocab"] - 1)
    alloc = dict(commit_min=2, tau_low=0.45, alpha0=1.0, beta0=1.0, kv_block=16, max_prompt=max(2, case["prompt_hi"]),
                 mode="sara", temperature=1.0, top_p=1.0, forced_eos_u32=0, prio_quant_bits=20, n_slots=case["slots"])
    if case["kind"] == "step":
        k = case["k"]
        alloc.update(B=case["groups"], k=k, n0=min(case["n0"], k), commit_min=k, budget_N=case["groups"] * k,
                     pool_U=case["pool"], max_new=case["max_new"], forced_eos_u32=FORCED_EOS)
    else:
        k = max(2, case["n0"])
        alloc.update(B=case["prompts"], k=k, n0=case["n0"], budget_N=case["prompts"] * k, pool_U=case["prompts"],
                     max_new=case["steps"] + 16, top_p=case["top_p"])
    return model, alloc


def _lengths(case, count):
    """The pool's prompt lengths: evenly over [prompt_lo, prompt_hi]."""
    lo, hi = case["prompt_lo"], case["prompt_hi"]
    return np.array([lo + (hi - lo) * i // max(1, count - 1) for i in range(count)], np.int64)


def _pool(case, alloc, seed):
    U, k, V = alloc["pool_U"], alloc["k"], case["vocab"]
    r = np.random.default_rng([int(seed), 2])
    off = np.zeros(U + 1, np.int32)
    off[1:] = np.cumsum(r.permutation(_lengths(case, U)))
    g = _gen(seed, 3)
    pool = dict(off=off, tokens=torch.randint(0, V - 1, (int(off[-1]),), generator=g, device="cuda", dtype=torch.int32),
                p=torch.rand(U, generator=g, device="cuda", dtype=torch.float64),
                forced=torch.randint(0, V - 1, (U * k, alloc["max_new"]), generator=g, device="cuda", dtype=torch.int32),
                forced_len=None)
    if case.get("ragged"):
        pool["forced_len"] = torch.randint(1, alloc["max_new"] + 1, (U * k,), generator=g, device="cuda", dtype=torch.int32)
    return pool


def prepare(case, seed):
    if case["kind"] == "sample":
        n, V, g = case["rows"], case["vocab"], _gen(seed, 4)
        i32 = dict(device="cuda", dtype=torch.int32)
        return dict(case=case, seed=seed, logits=torch.randn((n, V), generator=g, device="cuda") * 2.0,
                    rid=torch.randint(0, 4096, (n,), generator=g, **i32),
                    pos=torch.randint(0, 1024, (n,), generator=g, **i32), tok=torch.zeros(n, **i32))
    if case["kind"] == "predict":
        n, k, g = case["prompts"], case["k"], _gen(seed, 5)
        f64 = dict(device="cuda", dtype=torch.float64)
        done = torch.randint(0, k + 1, (n,), generator=g, device="cuda", dtype=torch.int32)
        good = (torch.rand(n, generator=g, **f64) * (done + 1)).to(torch.int32).clamp(max=done)
        good = torch.where(torch.rand(n, generator=g, **f64) < 0.6, torch.zeros_like(good), good)
        # warm-start priors Beta(1 + a, 1 + b) with fractional pseudo-counts
        alpha = 1.0 + 4.0 * torch.rand(n, generator=g, **f64)
        beta = 1.0 + 4.0 * torch.rand(n, generator=g, **f64)
        off = torch.arange(0, (case["groups"] + 1) * k, k, device="cuda", dtype=torch.int32)
        r = (torch.rand(case["groups"] * k, generator=g, device="cuda") < 0.4).float()
        return dict(case=case, alpha=alpha, beta=beta, n=done, s=good, out=torch.zeros(n, **f64), off=off, r=r,
                    adv=torch.zeros_like(r))
    model, alloc = _descs(case)
    w = [t.view(torch.int16) if t.dtype == torch.bfloat16 else t for t in _weights(case, seed)]
    ctx = sara.Sara(model, alloc, int(seed), w)
    pool = _pool(case, alloc, seed)
    logits = torch.zeros((case["slots"], case["vocab"]), dtype=torch.float32, device="cuda")
    return dict(case=case, ctx=ctx, pool=pool, logits=logits)


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    case = state["case"]
    if case["kind"] == "sample":
        f = sara.sara_sample_logits_noalloc if case["noalloc"] else sara.sara_sample_logits
        f(state["logits"], state["rid"], state["pos"], state["seed"], 3, case["temperature"], -1, 0, state["tok"],
          top_p=case["top_p"])
        return {"tokens": state["tok"]}
    if case["kind"] == "predict":
        sara.sara_peff_batch(state["alpha"], state["beta"], state["n"], state["s"], case["k"], state["out"])
        sara.grpo_group_advantages(state["r"], state["off"], 1e-6, state["adv"])
        return {"p_eff": state["out"], "adv": state["adv"]}
    ctx, pool = state["ctx"], state["pool"]
    ctx.sara_begin_step(pool["tokens"], pool["off"], pool["p"], pool["forced_len"], 0)
    if case["kind"] == "decode":
        if case["steps"]:
            ctx.sara_run(pool["forced"], graph_iters=16, max_iters=case["steps"])
        ctx.sara_decode_step(pool["forced"], state["logits"])
        return {"logits": state["logits"][:case["prompts"] * case["n0"]]}
    ctx.sara_decode_step(pool["forced"], state["logits"])
    ctx.sara_posterior_decide()
    ctx.sara_refill()
    ctx.sara_run(pool["forced"], graph_iters=16)
    ctx.sara_finish_step(1e-6)
    roll = ctx.read_rollouts()
    off, _, adv = ctx.read_advantages()
    # the committed groups' CSR, padded to the pool's size
    group_off = np.full(ctx.U + 1, off[-1], np.int32)
    group_off[:len(off)] = off
    out = {"logits": state["logits"], "p_eff": roll["p_eff"], "group_off": group_off,
           "adv": np.concatenate([adv, np.zeros(ctx.U * ctx.k - len(adv), np.float32)]),
           **{key: roll[key] for key in ("tokens", "length", "reward", "status", "n", "s")}}
    if case["dtype"] == "f32":      # in bf16 a last-bit change of the logits moves some draws
        out["sampled"] = roll["sampled"]
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    if case["kind"] == "sample":
        n, V = case["rows"], case["vocab"]
        return {"bytes": 4.0 * n * V + 12.0 * n, "flops": 60.0 * n * V}
    if case["kind"] == "predict":
        return {"bytes": 32.0 * case["prompts"] + (8.0 * case["k"] + 4.0) * case["groups"],
                "flops": 400.0 * case["prompts"] + 10.0 * case["k"] * case["groups"]}
    E = 2.0 if case["dtype"] == "bf16" else 4.0
    d, V, L = case["d"], case["vocab"], case["layers"]
    qd, kvd = case["hq"] * case["hd"], case["hkv"] * case["hd"]
    layer = L * (d * (qd + 2 * kvd) + qd * d + 3.0 * d * case["ffn"])       # layer weights
    head = 1.0 * V * d
    U = case["pool"] if case["kind"] == "step" else case["prompts"]
    P = _lengths(case, U).astype(np.float64)
    kv_tok = 2.0 * kvd * L * E                                             # K and V of one token
    # prefill of positions 0 .. P - 2
    pre = float(np.sum(P - 1))
    flops = 2.0 * layer * pre + 4.0 * qd * L * float(np.sum((P - 1) * P / 2))
    byts = layer * E * (pre > 0) + pre * (kv_tok + 2.0 * d * E)
    if case["kind"] == "step":
        # about n0 probes and two more rollouts a prompt in rounds of max_new tokens, over the drawn prompts
        drawn, rounds = min(case["groups"], U), 3
        rows, iters = drawn * min(case["n0"], case["k"]), rounds * case["max_new"]
    else:
        drawn, rows, iters = U, U * case["n0"], case["steps"] + 1
    mean_p = float(np.mean(P))
    for i in range(iters):
        gen = i % case["max_new"] if case["kind"] == "step" else i
        flops += 2.0 * (layer + head) * rows + 4.0 * qd * L * rows * (mean_p + gen)
        byts += (layer + head) * E + kv_tok * (drawn * (mean_p - 1) + rows * (gen + 1))
    return {"bytes": byts + 4.0 * rows * V, "flops": flops}


# ---------------------------------------------------------------------------
# tolerances, measured against exact()
# ---------------------------------------------------------------------------
def tolerance(case):
    if case["kind"] == "sample":
        return "exact"
    if case["kind"] == "predict":
        return {"rel": 1e-6}
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "differ": 0.002}
    # bf16 activations: the relative error of the logits grows with the depth
    return {"rel": 0.03 if case["layers"] > 4 else 0.02}


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _forward(case, w, seqs):
    """fp64 logits of the wanted positions of `seqs`: tuples (tokens, positions, mask, wanted)."""
    E = torch.float64
    hq, hkv, hd, L = case["hq"], case["hkv"], case["hd"], case["layers"]
    theta = 1.0e6 if case["dtype"] == "bf16" else 1.0e4
    inv = theta ** (-torch.arange(0, hd, 2, device="cuda", dtype=E) / hd)

    def norm(h, g):
        return h * torch.rsqrt((h * h).mean(-1, keepdim=True) + 1e-6) * g.to(E)

    def rope(x, c, s):
        a, b = x[..., :hd // 2], x[..., hd // 2:]
        return torch.cat([a * c - b * s, b * c + a * s], -1)

    hs = [w[0][tok].to(E) for tok, _, _, _ in seqs]
    for l in range(L):
        an, wq, wk, wv, wo, fn, wg, wu, wd = (t.to(E) for t in w[1 + 9 * l:10 + 9 * l])
        for i, (tok, pos, mask, _) in enumerate(seqs):
            T = len(tok)
            ang = pos.to(E)[:, None, None] * inv
            c, s = torch.cos(ang), torch.sin(ang)
            x = norm(hs[i], an)
            q = rope((x @ wq.T).view(T, hq, hd), c, s)
            kk = rope((x @ wk.T).view(T, hkv, hd), c, s)
            v = (x @ wv.T).view(T, hkv, hd)
            o = torch.empty(T, hq, hd, device="cuda", dtype=E)
            for h in range(hq):
                g = h // (hq // hkv)
                sc = (q[:, h].contiguous() @ kk[:, g].T.contiguous()) / math.sqrt(hd)
                o[:, h] = torch.softmax(sc.masked_fill(~mask, -math.inf), -1) @ v[:, g].contiguous()
            hs[i] = hs[i] + o.view(T, hq * hd) @ wo.T
            x = norm(hs[i], fn)
            hs[i] = hs[i] + (torch.nn.functional.silu(x @ wg.T) * (x @ wu.T)) @ wd.T
    x = norm(torch.cat([h[wanted] for h, (_, _, _, wanted) in zip(hs, seqs)]), w[1 + 9 * L])
    return x @ w[2 + 9 * L].to(E).T


def exact(case, seed):
    if case["kind"] == "sample":
        return None
    if case["kind"] == "predict":
        st = prepare(case, seed)
        k, n, s = case["k"], st["n"].double(), st["s"].double()
        a, b, r = st["alpha"] + s, st["beta"] + n - s, k - n
        lb = lambda x, y: torch.lgamma(x) + torch.lgamma(y) - torch.lgamma(x + y)  # noqa: E731
        zero = torch.zeros_like(a)
        sat = torch.where(s == 0, torch.exp(lb(a, b + r) - lb(a, b)), zero) + \
            torch.where(s == n, torch.exp(lb(a + r, b) - lb(a, b)), zero)
        pe = torch.where((s >= 1) & (n - s >= 1), torch.ones_like(a), torch.where(r <= 0, zero, 1.0 - sat))
        x = st["r"].double().view(case["groups"], k)
        adv = (x - x.mean(1, keepdim=True)) / (x.std(1, keepdim=True) + float(np.float32(1e-6)))
        return {"p_eff": pe, "adv": adv.view(-1)}
    if work(case)["flops"] > 3e14:
        return None
    _, alloc = _descs(case)
    pool, w, k = _pool(case, alloc, seed), _weights(case, seed), alloc["k"]
    if case["kind"] == "step":
        drawn = min(alloc["B"], alloc["budget_N"] // k, alloc["pool_U"])
        new = 0
    else:
        drawn, new = case["prompts"], case["steps"]
    off, n0 = pool["off"], alloc["n0"]
    rows = min(drawn * n0, case["slots"])
    seqs = []
    for u in range(-(-rows // n0)):
        # the prompt, then each rollout's generated tokens: a rollout attends to the prompt and to itself
        R = min(n0, rows - u * n0)
        P = int(off[u + 1] - off[u])
        tok = torch.cat([pool["tokens"][int(off[u]):int(off[u + 1])]] + [pool["forced"][u * k + j, :new] for j in range(R)])
        pos = torch.cat([torch.arange(P)] + [P + torch.arange(new)] * R).cuda()
        own = torch.cat([torch.full((P,), -1)] + [torch.full((new,), j) for j in range(R)]).cuda()
        mask = (pos[None, :] <= pos[:, None]) & ((own[None, :] < 0) | (own[None, :] == own[:, None]))
        wanted = [P - 1 + new * (j + 1) if new else P - 1 for j in range(R)]
        seqs.append((tok.long(), pos, mask, torch.tensor(wanted, device="cuda")))
    logits = _forward(case, w, seqs)
    if case["kind"] == "decode":
        return {"logits": logits}
    whole = torch.zeros((case["slots"], case["vocab"]), dtype=torch.float64, device="cuda")
    whole[:rows] = logits
    return {"logits": whole, "p_eff": None, "group_off": None, "adv": None, "tokens": None, "length": None,
            "reward": None, "status": None, "n": None, "s": None}
