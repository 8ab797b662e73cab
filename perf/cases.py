"""Performance cases: the calls that programs built on this library spend their time in.

Two paths, over the sizes that the workloads, the tests and the benchmark use:

* the LM-head objective.  ``lm_step`` is a training step (log-probabilities, a loss on them, dH and
  dW), ``lm_score`` the forward alone, for one or several weight matrices, with or without entropy;
* the KV-cache compression path.  ``kv_decode`` is what a decoding step adds to a cache, ``kv_gate`` the gate
  over a prompt, ``kv_cache`` the ragged store of gated states and their reconstruction, ``kv_train`` the gate's
  training pair (forward with its training outputs, then the backward).

Inputs are made on the GPU with the distributions of ``workloads/``; the references of ``exact`` are plain torch
in float64.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2603_04411_amd as L

VOCAB = 151936
CLIP, KL, EPS = 0.2, 0.04, 1e-6


def _lm(name, kind, P, G, T, d, V, dtype="bf16", lo=0.25, dist="uniform", loss="grpo", fp8=False, entropy=False,
        npol=1, dh16=False):
    """Response lengths lie in [lo * T, T]; `dist` is their distribution."""
    c = dict(kind=kind, P=P, G=G, T=T, d=d, V=V, dtype=dtype, lo=lo, dist=dist, loss=loss, fp8=fp8, entropy=entropy,
             npol=npol, dh16=dh16)
    return dict(c, name=name) if name else c


def _kv(name, kind, n, d, dtype="bf16", literal=False):
    c = dict(kind=kind, n=n, d=d, dtype=dtype, literal=literal)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The 2x4x32 fp32 workload, cross-entropy: unit runs and debugging, where launches and latency are all there is.
        _lm("step-f32-2x4x32", "lm_step", 2, 4, 32, 256, 4096, "f32", loss="ce"),
        # Scoring a few short completions of one prompt (a reward or rejection filter): some hundred tokens
        # against the whole vocabulary, bound by one read of W.
        _lm("score-8x24-d2048", "lm_score", 1, 8, 24, 2048, VOCAB),
        # The 8x8x256 workload: a small policy step.
        _lm("step-8x8x256-d2048", "lm_step", 8, 8, 256, 2048, VOCAB),
        # A micro-batch of the trajectory-balance workload: d = 3584, an odd number of slots per response, long-tailed
        # lengths.
        _lm("flowrl-4x16x500-d3584", "lm_step", 4, 16, 500, 3584, 152064, lo=1 / 128, dist="loguniform", loss="flowrl"),
        # Current, old and reference policy over the same hidden states with entropy, d = 5120 (two responses of
        # the 8x16x8192 workload).
        _lm("score3-1x2x8192-d5120", "lm_score", 1, 2, 8192, 5120, VOCAB, lo=0.125, entropy=True, npol=3),
        # A cross-entropy step with 8-bit logits and a bf16 dH.
        _lm("step-fp8-1x8x1024-d4096", "lm_step", 1, 8, 1024, 4096, VOCAB, loss="ce", fp8=True, dh16=True),
        # Four prompts of the 32x8x2048 workload: a micro-batch of the benchmarked step.
        _lm("step-4x8x2048-d4096", "lm_step", 4, 8, 2048, 4096, VOCAB),
        # A decoding step of 16 sequences appends one token each to a layer's key cache.
        _kv("kv-decode-16x1024", "kv_decode", 16, 1024),
        # The gate over the benchmark's stream: 16 prompts of 16K tokens, one layer.
        _kv("kv-gate-262144x1024", "kv_gate", 262144, 1024),
        # Store and reconstruction of one 16K-token sequence (an odd count: prompt plus what was decoded).
        _kv("kv-cache-16411x1024", "kv_cache", 16411, 1024),
        # Training the gate on one 4K-token sequence.
        _kv("kv-train-4096x1024", "kv_train", 4096, 1024),
        # The tests' small fp32 stream, Eq. 6 as printed.
        _kv("kv-train-f32-300x128", "kv_train", 300, 128, "f32", literal=True),
    ]


def _log_int(rng: random.Random, lo: float, hi: float) -> int:
    return max(int(lo), min(int(hi), int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    kind = rng.choice(["lm_step", "lm_step", "lm_score", "lm_score", "kv_decode", "kv_gate", "kv_cache", "kv_train"])
    if kind.startswith("lm"):
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        f32 = dtype == "f32"
        d = rng.choice([256, 320, 512, 1024] if f32 else [512, 768, 1024, 2048, 2560, 3584, 4096, 5120])
        V = _log_int(rng, 4000, 32768 if f32 else 152064)
        slots = _log_int(rng, 64, 4096 if f32 else 65536)
        # a drawn case stays below the largest listed one: fewer slots where V and d are large
        slots = min(slots, int(2.5e13 / (V * d * (16 if f32 else 1))))
        G = rng.choice([1, 2, 4, 7, 8, 16])
        P = rng.choice([1, 2, 3, 4, 8])
        T = max(4, slots // (P * G))
        step = kind == "lm_step"
        # over few tokens the surrogate's loss is a difference of nearly equal sums: no figure to compare by
        losses = ["grpo", "flowrl", "ce"] if P * G * T >= 4096 else ["flowrl", "ce"]
        return _lm(None, kind, P, G, T, d, V, dtype, lo=rng.choice([1 / 64, 0.125, 0.25, 1.0]),
                   dist=rng.choice(["uniform", "loguniform"]), loss=rng.choice(losses),
                   fp8=not f32 and d % 128 == 0 and rng.random() < 0.2, entropy=not step and rng.random() < 0.5,
                   npol=1 if step else rng.choice([1, 1, 2, 3]), dh16=step and not f32 and rng.random() < 0.3)
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    d = rng.choice([128, 256, 320, 512, 1024, 1024, 1024, 2048])
    n = {"kv_decode": lambda: _log_int(rng, 1, 256), "kv_gate": lambda: _log_int(rng, 256, 262144),
         "kv_cache": lambda: _log_int(rng, 256, 262144), "kv_train": lambda: _log_int(rng, 256, 65536)}[kind]()
    n = min(n, int((4 if dtype == "f32" else 16) * 2.0 ** 24 / d))
    return _kv(None, kind, n, d, dtype, literal=kind != "kv_cache" and rng.random() < 0.25)


# ---- inputs ------------------------------------------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _type(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _normal(g, rows, cols, std, dtype):
    """N(0, std^2) drawn in float32 and rounded to the storage type, in blocks of rows."""
    out = torch.empty(rows, cols, dtype=dtype, device="cuda")
    step = max(1, (1 << 28) // cols)
    for r in range(0, rows, step):
        m = min(step, rows - r)
        out[r:r + m] = torch.randn(m, cols, generator=g, device="cuda").mul_(std)
    return out


def _lengths(case, rng):
    T = case["T"]
    lo = max(1, int(case["lo"] * T))
    if case["dist"] == "uniform":
        return [rng.randint(lo, T) for _ in range(case["P"] * case["G"])]
    return [_log_int(rng, lo, T) for _ in range(case["P"] * case["G"])]


def _lm_inputs(case, seed):
    g, rng, dtype = _gen(seed), random.Random(seed), _type(case)
    P, G, T, d, V = (case[k] for k in ("P", "G", "T", "d", "V"))
    R, N = P * G, P * G * T
    lens = _lengths(case, rng)
    s = dict(H=_normal(g, N, d, 1.0, dtype))
    s["W"] = [_normal(g, V, d, 0.02, dtype) for _ in range(case["npol"])]
    # Zipf(1.1) token ids by inverting the distribution function; hot ids at the start of the vocabulary
    cdf = torch.arange(1, V + 1, dtype=torch.float64, device="cuda").pow_(-1.1).cumsum_(0)
    u = torch.rand(N, generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
    s["tok"] = torch.searchsorted(cdf, u, right=True).clamp_(max=V - 1).to(torch.int32)
    s["lens"] = torch.tensor(lens, dtype=torch.int32, device="cuda")
    if case["kind"] == "lm_step":
        if case["loss"] == "flowrl":
            s["reward"] = torch.rand(R, generator=g, device="cuda")
        else:
            s["reward"] = torch.tensor([float(rng.random() < 0.3) for _ in range(R)], device="cuda")
        s["logZ"] = torch.randn(P, generator=g, device="cuda")
        # The policy has moved a little from the one that sampled, along the advantages, and further from the
        # reference.  Its own log-probability is close to z_y - (ln V + |h|^2 std^2 / 2) for these weights.
        logp = torch.empty(N, device="cuda")
        for r in range(0, N, 8192):
            h = s["H"][r:r + 8192].float()
            z = (h * s["W"][0][s["tok"][r:r + 8192].long()].float()).sum(1)
            logp[r:r + 8192] = z - (math.log(V) + 0.5 * 0.02 ** 2 * h.square().sum(1))
        rw = s["reward"].view(P, G)
        adv = (rw - rw.mean(1, keepdim=True)) / (rw.std(1, keepdim=True, unbiased=False) + EPS)
        moved = adv.reshape(R, 1).expand(R, T).reshape(N)
        s["logp_old"] = logp - 0.05 * moved + 0.04 * torch.randn(N, generator=g, device="cuda")
        s["logp_ref"] = logp + 0.3 * torch.randn(N, generator=g, device="cuda")
    return s


def _fp8_exponent(t):
    """Largest power of two that keeps the largest magnitude below 224."""
    return int(math.floor(math.log2(224.0 / max(float(t.abs().max()), 1e-30))))


def _basis(d, seed):
    q, r = torch.linalg.qr(torch.randn(d, d, generator=torch.Generator().manual_seed(seed), dtype=torch.float32))
    return (q * r.diagonal().sign()).contiguous().cuda()     # q comes column by column


def _kv_inputs(case, seed):
    g, dtype = _gen(seed), _type(case)
    n, d = case["n"], case["d"]
    s = {}
    sigma = torch.arange(1, d + 1, dtype=torch.float32, device="cuda").pow(-0.5)
    if case["kind"] == "kv_cache":
        # spectral states and retained counts as the gate leaves them: a mean of 0.44 d, spread 0.11 d
        s["xt"] = torch.empty(n, d, dtype=dtype, device="cuda")
        for r in range(0, n, 65536):
            m = min(65536, n - r)
            s["xt"][r:r + m] = torch.randn(m, d, generator=g, device="cuda") * sigma
        k = (0.44 + 0.11 * torch.randn(n, generator=g, device="cuda")) * d
        s["k"] = k.round_().clamp_(1, d).to(torch.int32)
        s["U_inv"] = _basis(d, seed).t().contiguous().to(dtype)
        return s
    Q = _basis(d, seed)
    s["x"] = torch.empty(n, d, dtype=dtype, device="cuda")
    for r in range(0, n, 65536):
        m = min(65536, n - r)
        s["x"][r:r + m] = (torch.randn(m, d, generator=g, device="cuda") * sigma) @ Q.t()
    s["U"] = (Q + 0.02 / math.sqrt(d) * torch.randn(d, d, generator=g, device="cuda")).to(dtype)
    s["W"] = (1.5 * torch.randn(d, d, generator=g, device="cuda")).to(dtype)
    j = torch.arange(d, dtype=torch.float32, device="cuda")
    s["b"] = 6.0 * torch.exp(-((j - 0.35 * d) ** 2) / (2 * (0.12 * d) ** 2))
    if case["kind"] == "kv_train":
        s["g_xhat"] = _normal(g, n, d, 1.0 / math.sqrt(n), dtype)
    return s


TAU, ALPHA = 0.1, 0.5
CACHE_TOKENS = 64      # tokens that a decoding case's cache already holds (at a retain rate of one half)


def _mask_grad(case):
    """Gradient of the regulariser on every mask element, 2 alpha R / (n d), at a running mean R of 0.44."""
    return 2 * ALPHA * 0.44 / (case["n"] * case["d"])


def prepare(case, seed):
    f32 = dict(dtype=torch.float32, device="cuda")
    i32 = dict(dtype=torch.int32, device="cuda")
    dtype = _type(case)
    if case["kind"].startswith("lm"):
        s = _lm_inputs(case, seed)
        P, G, T, d, V = (case[k] for k in ("P", "G", "T", "d", "V"))
        R, N = P * G, P * G * T
        flags = (L.binding.FLAG_FP8_LOGITS if case["fp8"] else 0) | (L.binding.FLAG_DH_BF16 if case["dh16"] else 0)
        exps = {}
        if case["fp8"]:
            exps = dict(fp8_exp_h=_fp8_exponent(s["H"]), fp8_exp_w=min(_fp8_exponent(w) for w in s["W"]))
        s["desc"] = L.make_desc(P, G, T, d, V, case["dtype"], flags=flags, **exps)
        nbytes = L.multi_workspace_bytes(s["desc"], case["npol"])
        s["ws"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        s["logp"] = [torch.empty(N, **f32) for _ in range(case["npol"])]
        s["lse"] = torch.empty(N, **f32)
        s["entropy"] = torch.empty(N, **f32) if case["entropy"] else None
        s["mask"], s["cu_len"] = torch.empty(N, dtype=torch.uint8, device="cuda"), torch.empty(R + 1, **i32)
        if case["kind"] == "lm_step":
            s["adv"], s["loss"], s["stats"] = torch.empty(R, **f32), torch.empty(1, **f32), torch.empty(4, **f32)
            s["g_logZ"], s["resid"], s["g_logp"] = torch.empty(P, **f32), torch.empty(R, **f32), torch.empty(N, **f32)
            s["dH"] = torch.empty(N, d, dtype=torch.bfloat16 if case["dh16"] else torch.float32, device="cuda")
            s["dW"] = torch.empty(V, d, **f32)
            nbytes = max(L.loss_workspace_bytes(P, G, T), L.loss_workspace_bytes(R, 1, T))
            s["loss_ws"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    else:
        s = _kv_inputs(case, seed)
        n, d = case["n"], case["d"]
        s["desc"] = L.make_kv_desc(n, d, case["dtype"], flags=L.FLAG_LITERAL_FLIP if case["literal"] else 0)
        s["ws"] = torch.empty(L.dynakv_workspace_bytes(s["desc"]), dtype=torch.uint8, device="cuda")
        base = 8 * (CACHE_TOKENS * d // 16) if case["kind"] == "kv_decode" else 0
        if case["kind"] != "kv_cache":
            s["xt"], s["k"] = torch.empty(n, d, dtype=dtype, device="cuda"), torch.empty(n, **i32)
        if case["kind"] in ("kv_decode", "kv_cache"):
            s["base"] = base
            s["off"] = torch.empty(n + 1, dtype=torch.int64, device="cuda")
            s["packed"] = torch.zeros(base + n * d, dtype=dtype, device="cuda")
        if case["kind"] == "kv_cache":
            s["xbar"] = torch.empty(n, d, dtype=dtype, device="cuda")
        if case["kind"] == "kv_train":
            s["m"], s["xhat"] = torch.empty(n, d, **f32), torch.empty(n, d, dtype=dtype, device="cuda")
            s["retain"] = torch.empty(3, **f32)
            s["dx"] = torch.empty(n, d, dtype=dtype, device="cuda")
            s["dU"], s["dW"], s["db"] = torch.empty(d, d, **f32), torch.empty(d, d, **f32), torch.empty(d, **f32)
            s["bws"] = torch.empty(L.dynakv_bwd_workspace_bytes(s["desc"]), dtype=torch.uint8, device="cuda")
    s["case"] = case
    return s


# ---- one pass ----------------------------------------------------------------------------------------------


def run(s):
    case = s["case"]
    return {"lm_step": _run_lm_step, "lm_score": _run_lm_score, "kv_decode": _run_kv_decode, "kv_gate": _run_kv_gate,
            "kv_cache": _run_kv_cache, "kv_train": _run_kv_train}[case["kind"]](s, case)


def _run_lm_score(s, case):
    if case["npol"] == 1:
        L.lmhead_logprob_fwd(s["desc"], s["H"], s["W"][0], s["tok"], s["lens"], s["logp"][0], s["lse"], s["entropy"],
                             s["mask"], s["cu_len"], s["ws"])
    else:
        L.lmhead_logprob_fwd_multi(s["desc"], s["H"], s["W"], s["tok"], s["lens"], s["logp"], s["lse"], s["entropy"],
                                   s["mask"], s["cu_len"], s["ws"])
    return dict(logp=s["logp"], lse=s["lse"], entropy=s["entropy"], mask=s["mask"], cu_len=s["cu_len"])


def _run_lm_step(s, case):
    P, G, T = case["P"], case["G"], case["T"]
    out = _run_lm_score(s, case)
    if case["loss"] == "flowrl":
        L.flowrl_tb_loss(s["logp"][0], s["logp_ref"], s["reward"], s["logZ"], s["lens"], P, G, T, 15.0, s["loss"],
                         s["g_logp"], s["g_logZ"], s["resid"], s["loss_ws"])
        out.update(g_logZ=s["g_logZ"], resid=s["resid"])
    elif case["loss"] == "ce":
        L.ce_loss(s["logp"][0], s["lens"], P * G, T, s["loss"], s["g_logp"], s["loss_ws"])
    else:
        L.group_advantage(s["reward"], P, G, EPS, 0, s["adv"])
        L.grpo_loss(s["logp"][0], s["logp_old"], s["logp_ref"], s["adv"], s["lens"], P, G, T, CLIP, CLIP, KL, 0,
                    s["loss"], s["g_logp"], s["stats"], s["loss_ws"])
        out.update(adv=s["adv"], stats=s["stats"])
    L.lmhead_logprob_bwd(s["desc"], s["H"], s["W"][0], s["tok"], s["lens"], s["lse"], s["g_logp"], s["dH"], s["dW"],
                         s["ws"])
    out.update(loss=s["loss"], g_logp=s["g_logp"], dH=s["dH"], dW=s["dW"])
    return out


def _run_kv_decode(s, case):
    L.dynakv_gate(s["desc"], s["x"], s["U"], s["W"], s["b"], TAU, s["xt"], s["k"], None, None, s["ws"])
    L.dynakv_store(s["desc"], s["xt"], s["k"], s["base"], s["off"], s["packed"], s["packed"].numel(), s["ws"])
    return dict(xt=s["xt"], k=s["k"], off=s["off"], packed=s["packed"])


def _run_kv_gate(s, case):
    L.dynakv_gate(s["desc"], s["x"], s["U"], s["W"], s["b"], TAU, s["xt"], s["k"], None, None, s["ws"])
    return dict(xt=s["xt"], k=s["k"])


def _run_kv_cache(s, case):
    L.dynakv_store(s["desc"], s["xt"], s["k"], s["base"], s["off"], s["packed"], s["packed"].numel(), s["ws"])
    L.dynakv_reconstruct(s["desc"], s["packed"], s["packed"].numel(), s["off"], s["k"], s["U_inv"], s["xbar"], s["ws"])
    return dict(off=s["off"], packed=s["packed"], xbar=s["xbar"])


def _run_kv_train(s, case):
    L.dynakv_gate(s["desc"], s["x"], s["U"], s["W"], s["b"], TAU, s["xt"], s["k"], s["m"], s["xhat"], s["ws"])
    L.dynakv_retain(s["desc"], s["k"], s["m"], ALPHA, s["retain"], None, s["ws"])
    L.dynakv_gate_bwd(s["desc"], s["x"], s["U"], s["W"], s["b"], s["xt"], s["g_xhat"], None, _mask_grad(case), s["dx"],
                      s["dU"], s["dW"], s["db"], s["bws"])
    return dict(xt=s["xt"], k=s["k"], m=s["m"], xhat=s["xhat"], retain=s["retain"], dx=s["dx"], dU=s["dU"],
                dW=s["dW"], db=s["db"])


# ---- what a pass cannot do without -------------------------------------------------------------------------


def work(case):
    esz = 2 if case["dtype"] == "bf16" else 4
    if case["kind"].startswith("lm"):
        P, G, T, d, V, npol = (case[k] for k in ("P", "G", "T", "d", "V", "npol"))
        lo = max(1, int(case["lo"] * T))
        mean = (lo + T) / 2 if case["dist"] == "uniform" or lo == T else (T - lo) / math.log(T / lo)
        N, nv = P * G * T, P * G * mean
        # valid rows of H, W, token ids, lengths; log-probabilities, lse, entropy, mask, offsets
        nbytes = nv * d * esz + npol * V * d * esz + 4 * nv + 4 * N * (npol + 1 + case["entropy"]) + N + 8 * P * G
        flops = 2.0 * nv * V * d * npol
        if case["kind"] == "lm_step":
            nbytes += 8 * nv + 4 * N + N * d * (2 if case["dh16"] else 4) + 4 * V * d   # old and ref, g_logp, dH, dW
            flops *= 3
        return {"bytes": nbytes, "flops": flops}
    n, d, kind = case["n"], case["d"], case["kind"]
    if kind == "kv_cache":
        kept = 0.44 * n * d
        return {"bytes": (3 * kept + n * d + d * d) * esz + 12 * n, "flops": 2.0 * kept * d}
    nbytes = (2 * n * d + 2 * d * d) * esz + 4 * d + 4 * n
    flops = 4.0 * n * d * d
    if kind == "kv_decode":
        nbytes += 0.5 * n * d * esz + 8 * n
    if kind == "kv_train":
        nbytes += n * d * (3 * esz + 4) + 8 * d * d + 4 * d     # xhat, g_xhat, dx, m; dU, dW, db
        flops += 8.0 * n * d * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Differences come from the order of fp32 sums and, in bf16, from where they are rounded next (dZ, the spectral
    # state, the gate's gradients).
    if case["kind"] == "kv_cache":
        return {"rel": 8e-3} if case["dtype"] == "bf16" else {"rel": 1e-5}
    if case["dtype"] == "f32":
        return {"rel": 2e-5, "differ": 0.005} if case["kind"].startswith("kv") else {"rel": 2e-5}
    if case["kind"] == "lm_score":
        return {"rel": 1e-5}
    if case["kind"] == "lm_step":
        return {"rel": 8e-3}
    return {"rel": 1.2e-2, "differ": 0.005}


# ---- references in 64 bits ---------------------------------------------------------------------------------


def exact(case, seed):
    if case["kind"].startswith("lm"):
        return _exact_lm(case, seed)
    s = _kv_inputs(case, seed)
    return _exact_kv_cache(case, s) if case["kind"] == "kv_cache" else _exact_kv(case, s)


def _e4m3(t, e):
    return (t.float() * 2.0 ** e).clamp_(-448, 448).to(torch.float8_e4m3fn).double() * 2.0 ** -e


def _exact_lm(case, seed):
    s = _lm_inputs(case, seed)
    P, G, T, V = (case[k] for k in ("P", "G", "T", "V"))
    R, N = P * G, P * G * T
    valid = (torch.arange(T, device="cuda")[None, :] < s["lens"][:, None].long()).reshape(N)
    rows = valid.nonzero().flatten()
    tok = s["tok"].long()[rows]
    Hv = s["H"][rows].double()
    if case["fp8"]:
        eh, ew = _fp8_exponent(s["H"]), min(_fp8_exponent(w) for w in s["W"])
        Hz = _e4m3(s["H"][rows], eh)
        weight = lambda p, a, b: _e4m3(s["W"][p][a:b], ew)  # noqa: E731
    else:
        Hz = Hv
        weight = lambda p, a, b: s["W"][p][a:b].double()  # noqa: E731
    step = max(256, (1 << 28) // max(1, rows.numel()))
    spread = lambda v: torch.zeros(N, dtype=torch.float64, device="cuda").index_copy_(0, rows, v)  # noqa: E731

    logps, lse0, ent0 = [], None, None
    for p in range(case["npol"]):
        m = torch.full_like(Hz[:, 0], -math.inf)
        t1, t2, zy = torch.zeros_like(m), torch.zeros_like(m), torch.zeros_like(m)
        for a in range(0, V, step):
            b = min(V, a + step)
            z = Hz @ weight(p, a, b).t()
            here = (tok >= a) & (tok < b)
            zy = torch.where(here, z.gather(1, (tok - a).clamp(0, b - a - 1)[:, None])[:, 0], zy)
            mn = torch.maximum(m, z.amax(1))
            scale = (m - mn).exp()
            e = (z - mn[:, None]).exp_()
            t1 = t1 * scale + e.sum(1)
            if case["entropy"] and p == 0:
                t2 = t2 * scale + e.mul_(z).sum(1)
            m = mn
        lse = m + t1.log()
        logps.append(spread(zy - lse))
        if p == 0:
            lse0, ent0 = lse, lse - t2 / t1
    out = dict(logp=logps, lse=spread(lse0), entropy=spread(ent0) if case["entropy"] else None, mask=None, cu_len=None)
    if case["kind"] == "lm_score":
        return out

    logp = logps[0].view(R, T)
    ok, n = valid.view(R, T), s["lens"].double()
    if case["loss"] == "flowrl":
        mean = lambda v: torch.where(ok, v.double().view(R, T), 0.0).sum(1) / n  # noqa: E731
        delta = s["logZ"].double().repeat_interleave(G) - 15.0 * s["reward"].double() + mean(logp) - mean(s["logp_ref"])
        loss = delta.square().mean().view(1)
        g = torch.where(ok, (2 * delta / (R * n))[:, None], 0.0)
        out.update(g_logZ=2.0 / R * delta.view(P, G).sum(1), resid=delta)
    elif case["loss"] == "ce":
        loss = -(torch.where(ok, logp, 0.0).sum() / n.sum()).view(1)
        g = torch.where(ok, -1.0 / n.sum(), 0.0)
    else:
        rw = s["reward"].double().view(P, G)
        adv = ((rw - rw.mean(1, keepdim=True)) / (rw.std(1, keepdim=True, unbiased=False) + EPS)).reshape(R)
        A = adv[:, None]
        rho = (logp - s["logp_old"].double().view(R, T)).exp()
        dl = s["logp_ref"].double().view(R, T) - logp
        k3 = dl.exp() - dl - 1
        free = torch.where(A >= 0, rho <= 1 + CLIP, rho >= 1 - CLIP)
        w = torch.where(ok, 1.0 / (R * n[:, None]), 0.0)
        surr = torch.minimum(rho * A, rho.clamp(1 - CLIP, 1 + CLIP) * A)
        loss = (w * (KL * k3 - surr)).sum().view(1)
        g = w * (torch.where(free, -A * rho, 0.0) + KL * (1 - dl.exp()))
        total = n.sum()
        stats = [(ok & ~free).sum().double(), torch.where(ok, k3, 0.0).sum(), torch.where(ok, rho, 0.0).sum()]
        out.update(adv=adv, stats=torch.stack([v / total for v in stats] + [total]))
    gv = g.reshape(N)[rows]
    dH = torch.zeros(N, case["d"], dtype=torch.float64, device="cuda")
    dW = torch.empty(V, case["d"], dtype=torch.float64, device="cuda")
    acc = torch.zeros_like(Hv)
    for a in range(0, V, step):
        b = min(V, a + step)
        dz = (Hz @ weight(0, a, b).t()).sub_(lse0[:, None]).exp_().neg_()
        here = ((tok >= a) & (tok < b)).nonzero().flatten()
        dz[here, tok[here] - a] += 1.0
        dz.mul_(gv[:, None])
        acc += dz @ s["W"][0][a:b].double()
        dW[a:b] = dz.t() @ Hv
    dH[rows] = acc
    out.update(loss=loss, g_logp=g.reshape(N), dH=dH, dW=dW)
    return out


def _exact_kv_cache(case, s):
    n, d = case["n"], case["d"]
    k = s["k"].long()
    seg = (k + 7) // 8 * 8
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    off[1:] = seg.cumsum(0)
    packed = torch.zeros(n * d, dtype=s["xt"].dtype, device="cuda")
    xbar = torch.empty(n, d, dtype=torch.float64, device="cuda")
    j = torch.arange(d, device="cuda")
    Ui = s["U_inv"].double()
    for r in range(0, n, 32768):
        e = min(n, r + 32768)
        keep = j[None, :] < k[r:e, None]
        packed[(off[r:e, None] + j)[keep]] = s["xt"][r:e][keep]
        xbar[r:e] = torch.where(keep, s["xt"][r:e].double(), 0.0) @ Ui
    return dict(off=off, packed=packed, xbar=xbar)


def _exact_kv(case, s):
    """The gate in 64 bits throughout (the library rounds the spectral state to the storage type)."""
    n, d, train = case["n"], case["d"], case["kind"] == "kv_train"
    U, W, b = s["U"].double(), s["W"].double(), s["b"].double()
    flip = (lambda t: t.flip(1)) if case["literal"] else (lambda t: t)     # gate columns <-> mask positions
    xt = torch.empty(n, d, dtype=torch.float64, device="cuda")
    out = dict(xt=xt, k=None)
    if case["kind"] == "kv_decode":
        out.update(off=None, packed=None)
    if train:
        m, xhat, dx = torch.empty_like(xt), torch.empty_like(xt), torch.empty_like(xt)
        dU, dW, db = torch.zeros_like(U), torch.zeros_like(U), torch.zeros_like(b)
    kept = 0
    for r in range(0, n, 16384):
        e = min(n, r + 16384)
        x = s["x"][r:e].double()
        xt[r:e] = x @ U
        if not train:
            continue
        p = flip(torch.softmax(xt[r:e] @ W + b, 1))
        m[r:e] = p.flip(1).cumsum(1).flip(1)
        xhat[r:e] = xt[r:e] * m[r:e]
        kept += int((m[r:e].float() > TAU).sum())
        gx = s["g_xhat"][r:e].double()
        q = (gx * xt[r:e] + _mask_grad(case)).cumsum(1)
        gl = flip(p * (q - (p * q).sum(1, keepdim=True)))
        gxt = gx * m[r:e] + gl @ W.t()
        dx[r:e] = gxt @ U.t()
        dU += x.t() @ gxt
        dW += xt[r:e].t() @ gl
        db += gl.sum(0)
    if train:
        soft = m.mean()
        retain = torch.stack([soft.new_tensor(kept / (n * d)), soft, ALPHA * soft ** 2])
        out.update(m=m, xhat=xhat, retain=retain, dx=dx, dU=dU, dW=dW, db=db)
    return out
