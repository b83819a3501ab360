"""Timed cases of the pruning path: what a program that uses the library runs.

Every case goes through the public entry points of paper_2609_37581_amd.trevs
with the handles (outputs and workspace allocated once) that a serving program
keeps.  A case is a dict of plain values; `kind` names the entry point:

  prellm     stage 1, before the LLM: trevs.Prellm (k_div > 0 adds the
             farthest-point diversity set, the paper's K_r : K_d = 3 : 1)
  inllm      stage 2, at one LLM layer: trevs.Inllm
  analysis   the diagnostics of two questions about one image:
             trevs.TextSensitivity, then trevs.TopkSpearman on the scores

Sizes are those of the workloads in synthetic/workloads.py (LLaVA-1.5-7B,
LLaVA-NeXT-7B and Qwen2.5-VL-7B shapes) and generic odd ones.
"""

import math

import torch

from paper_2609_37581_amd import trevs

PREFIX = 35  # chat-template rows before the visual block

# ----------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------


def _prellm(name, **kw):
    c = dict(name=name, kind="prellm", dtype="bf16", n_seg=1, H_v=16, ragged=False, k_div=0,
             mode="weights", rho=0.5)
    c.update(kw)
    return c


def _inllm(name, **kw):
    c = dict(name=name, kind="inllm", dtype="bf16", P=PREFIX, d_h=128, n_pos=1, ragged=False,
             softmax="visual")
    c.update(kw)
    return c


def listed():
    return [
        # one image of an interactive chat in fp32: launches and latency
        _prellm("s1-llava15-b1-f32", dtype="f32", B=1, N=576, d=4096, M=32, K=192),
        # a served batch of single images, questions of 16 to 64 tokens
        _prellm("s1-llava15-b64", B=64, N=576, d=4096, M=64, ragged=True, K=192),
        # a batch of multi-tile images, softmax per tile
        _prellm("s1-llavanext-b16", B=16, N=2880, n_seg=5, d=4096, M=64, K=640),
        # long visual sequences (high resolution or video): the benchmark's stage 1
        _prellm("s1-qwen-b4", B=4, N=16384, d=3584, M=128, K=4096),
        # odd sizes in fp32, budget split between the two scores: the analysis
        # of a textual ratio on a 37 x 37 patch grid
        _prellm("s1-odd-b3-f32-budget", dtype="f32", B=3, N=1369, d=1152, M=77, ragged=True, K=457,
                mode="budget", rho=0.25),
        # with the diversity set, as the paper prunes: multi-tile images
        _prellm("s1-div-llavanext-b16", B=16, N=2880, n_seg=5, d=4096, M=64, K=640, k_div=160),
        # with the diversity set on long visual sequences: the largest call
        _prellm("s1-div-qwen-b4", B=4, N=16384, d=3584, M=128, K=4096, k_div=1024),
        # stage 2 of one image of an interactive chat in fp32
        _inllm("s2-llava15-b1-f32", dtype="f32", B=1, K_in=192, T=32, H_q=32, H_kv=32, D=4096,
               n_keep=8, K=32),
        # stage 2 of a served batch, ragged questions
        _inllm("s2-llava15-b64", B=64, K_in=192, T=64, ragged=True, H_q=32, H_kv=32, D=4096,
               n_keep=16, K=64),
        # odd sizes, grouped-query heads, the layer's own causal softmax
        _inllm("s2-odd-b5-causal", B=5, K_in=637, T=45, ragged=True, H_q=32, H_kv=8, D=4096,
               n_keep=16, K=213, softmax="causal"),
        # stage 2 of long visual sequences with M-RoPE position planes
        _inllm("s2-qwen-b4", B=4, K_in=4096, T=128, H_q=28, H_kv=4, D=3584, n_keep=14, K=1024, n_pos=3),
        # head sensitivity of two questions about each image, and the rank
        # correlation of the two scores
        dict(name="analysis-qwen-b4", kind="analysis", dtype="bf16", B=4, N=16384, K_in=4096, T=128,
             ragged=False, P=PREFIX, H_q=28, H_kv=4, d_h=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("prellm", "prellm", "prellm", "div", "div", "inllm", "inllm", "inllm", "analysis"))
    dtype = rng.choice(("bf16", "bf16", "bf16", "f32"))
    ragged = rng.random() < 0.5
    if kind in ("prellm", "div"):
        d = rng.choice((1024, 1152, 2048, 3584, 4096, 4104, 5120))
        seg = rng.choice((1, 1, 5))
        N = seg * _log_int(rng, max(1, 256 // seg), 16384 // seg)
        B = _log_int(rng, 1, max(1, min(64, 65536 // N)))
        M = rng.randint(12, 128)
        K = max(4, int(N * rng.choice((0.5, 0.25, 1 / 3, 1 / 9))))
        c = dict(kind="prellm", dtype=dtype, B=B, N=N, n_seg=seg, H_v=16, d=d, M=M, ragged=ragged, K=K,
                 k_div=0, mode="weights", rho=rng.choice((0.25, 0.5, 0.5, 0.75)))
        if kind == "div":
            if B * N * N * d > 4 * 16384 * 16384 * 3584:  # no more work than the largest listed call
                c["B"] = B = max(1, B // 2)
            if dtype == "f32":  # the matrix cores multiply fp32 at a fraction of the bf16 rate
                c["N"] = N = seg * max(1, min(N, 4096) // seg)
                c["K"] = K = max(4, min(K, N // 3))
                c["B"] = min(B, 4)
            c["k_div"] = max(1, min(K // 4, 1024))
        elif rng.random() < 0.25:
            c["mode"] = "budget"
        return c
    heads = rng.choice(((32, 32, 128), (28, 4, 128), (32, 8, 128), (16, 16, 64), (8, 1, 256)))
    K_in = _log_int(rng, 64, 4096)
    B = _log_int(rng, 1, max(1, min(64, 16384 // K_in)))
    T = rng.randint(12, 128)
    if kind == "analysis":
        return dict(kind="analysis", dtype=dtype, B=B, N=4 * K_in, K_in=K_in, T=T, ragged=ragged,
                    P=rng.randint(1, 64), H_q=heads[0], H_kv=heads[1], d_h=heads[2])
    return dict(kind="inllm", dtype=dtype, B=B, K_in=K_in, T=T, ragged=ragged, P=rng.randint(0, 64),
                H_q=heads[0], H_kv=heads[1], d_h=heads[2], D=rng.choice((2048, 3584, 4096)),
                n_keep=heads[0] // 2, K=max(1, int(K_in * rng.choice((1 / 3, 1 / 4, 1 / 6)))),
                n_pos=rng.choice((1, 1, 3)), softmax=rng.choice(("visual", "causal")))


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------


class _Draws:
    """Random tensors on the GPU (and small integers on the host), from the seed alone."""

    def __init__(self, case, seed):
        self.dev = torch.device("cuda")
        self.gen = torch.Generator(self.dev).manual_seed(seed & 0x7fffffff)
        self.host = torch.Generator().manual_seed(seed & 0x7fffffff)
        self.dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16

    def normal(self, *shape):
        return torch.randn(shape, generator=self.gen, device=self.dev, dtype=torch.float32)

    def lengths(self, B, hi, ragged):
        if not ragged:
            return None
        return torch.randint(max(1, hi // 4), hi + 1, (B,), generator=self.host).to(self.dev, torch.int32)

    def some(self, n, k):
        return torch.randperm(n, generator=self.host)[:k].to(self.dev)


def _stage1(c, seed):
    """[CLS] logits ~ N(0,1), raised by 4 in every head at a few salient
    patches.  Visual features as images give them: a direction shared by all
    tokens, one per image region (runs of neighbouring tokens), and the
    token's own; a few query-matched tokens at cosine 0.6 to the mean text
    direction.  Text rows ~ N(0, 1/d), zero past their length."""
    r = _Draws(c, seed)
    B, N, d, M = c["B"], c["N"], c["d"], c["M"]
    cls = r.normal(B, c["H_v"], N)
    Z = torch.empty((B, N, d), device=r.dev, dtype=r.dt)
    T = r.normal(B, M, d) / math.sqrt(d)
    tl = r.lengths(B, M, c["ragged"])
    if tl is not None:
        T *= (torch.arange(M, device=r.dev)[None, :] < tl[:, None])[:, :, None]
    few = max(1, N // 64)
    regions = torch.arange(N, device=r.dev) // 24
    for b in range(B):
        order = r.some(N, 2 * few)
        cls[b][:, order[:few]] += 4.0
        z = r.normal(N, d)
        z *= 0.8
        z += 0.5 * r.normal(int(regions[-1]) + 1, d)[regions]
        z += 0.33 * r.normal(1, d)
        u = T[b].sum(0)
        u = u / u.norm()
        g = z[order[few:]]
        g = g - (g @ u)[:, None] * u
        norm = g.norm(dim=1, keepdim=True)
        z[order[few:]] = norm * (0.6 * u + 0.8 * g / norm)
        Z[b] = (z / math.sqrt(d)).to(r.dt)
    return cls.to(r.dt), Z, T.to(r.dt), tl


def _queries(r, c, S, beta, base=None):
    """Query rows ~ N(0,1) scaled per head (0.5 to 2); a quarter of the heads
    see a direction shared with some visual key rows."""
    q = r.normal(c["B"], S, c["H_q"], c["d_h"]) if base is None else base + 0.1 * r.normal(*base.shape)
    return q * beta[:, None] if base is None else q


def _stage2(c, seed, questions=1):
    r = _Draws(c, seed)
    B, P, K, H, G = c["B"], c["P"], c["K_in"], c["H_q"], c["H_q"] // c["H_kv"]
    S = P + K + c["T"]
    beta = torch.linspace(0.5, 2.0, H, device=r.dev)[r.some(H, H)]
    k = r.normal(B, S, c["H_kv"], c["d_h"])
    sens = r.some(H, max(1, H // 4))
    qs, base = [], None
    for _ in range(questions):
        rows = r.some(K, max(1, K // 8))
        way = r.normal(c["H_kv"], c["d_h"])
        way *= math.sqrt(3.0 * math.sqrt(c["d_h"])) / way.norm(dim=1, keepdim=True)
        k[:, P + rows] += way
        base = q = _queries(r, c, S, beta, base)
        q = q.clone()
        q[:, P + K:, sens] += way[sens // G]
        qs.append(q.to(r.dt))
    lens = [r.lengths(B, c["T"], c["ragged"]) for _ in range(questions)]
    return r, S, qs, k.to(r.dt), lens


def prepare(case, seed):
    c = case
    if c["kind"] == "prellm":
        cls, Z, T, tl = _stage1(c, seed)
        return trevs.Prellm(cls, Z, T, tl, k_keep=c["K"], n_seg=c["n_seg"], k_div=c["k_div"],
                            textual_ratio=c["rho"], want_scores=True, ratio_mode=c["mode"])
    if c["kind"] == "inllm":
        r, S, (q,), k, (tl,) = _stage2(c, seed)
        v = r.normal(c["B"], S, c["H_kv"], c["d_h"]).to(r.dt)
        hidden = r.normal(c["B"], S, c["D"]).to(r.dt)
        pos = torch.arange(S, device=r.dev).expand(c["n_pos"], c["B"], S).contiguous()
        return trevs.Inllm(q, k, v, hidden, pos, tl, P=c["P"], K_in=c["K_in"], n_keep_heads=c["n_keep"],
                           k_keep=c["K"], want_scores=True, softmax=c["softmax"])
    r, S, (q0, q1), k, (t0, t1) = _stage2(c, seed, questions=2)
    sv = torch.softmax(r.normal(c["B"], 16, c["N"]), dim=2).mean(1)
    st = (1.0 + 0.1 * r.normal(c["B"], c["N"])).abs() / math.sqrt(2 * 3584)
    return (trevs.TextSensitivity(q0, k, q1, k, t0, t1, P=c["P"], K_in=c["K_in"]),
            trevs.TopkSpearman(sv, st, c["N"] // 4))


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------


def run(state):
    if isinstance(state, trevs.Prellm):
        idx, feats = state()
        return dict(idx=idx, feats=feats, div=state.div_idx, score=state.score, sal=state.sal,
                    rel=state.rel, norm=state.norm_stats)
    if isinstance(state, trevs.Inllm):
        idx, hidden, k, v, pos = state()
        return dict(idx=idx, hidden=hidden, k=k, v=v, pos=pos, heads=state.head_sel, var=state.head_var,
                    score=state.score)
    sens, spear = state
    ts = sens()
    rho, idx = spear()
    return dict(ts=ts, p0=sens.profile[0], p1=sens.profile[1], v0=sens.head_var[0], v1=sens.head_var[1],
                rho=rho, idx=idx)


def work(case):
    """Every input read once, every output written once; the products that no
    order of the steps saves."""
    c = case
    e = 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "prellm":
        B, N, d, K = c["B"], c["N"], c["d"], c["K"]
        M = c["M"] * (0.625 if c["ragged"] else 1.0)
        scores = 2 if c["mode"] == "budget" else 3
        # with a diversity set every token meets every selected token once
        pairs = N * (M + (K if c["k_div"] else 0))
        return dict(bytes=B * (c["H_v"] * N * e + N * d * e + M * d * e + K * d * e + K * 4 + scores * N * 4),
                    flops=2.0 * B * pairs * d)
    B, P, K_in = c["B"], c["P"], c["K_in"]
    T = c["T"] * (0.625 if c["ragged"] else 1.0)
    q, kv = c["H_q"] * c["d_h"] * e, c["H_kv"] * c["d_h"] * e
    flops = 2.0 * B * T * K_in * c["H_q"] * c["d_h"]
    if c["kind"] == "inllm":
        S_out = P + c["K"] + c["T"]
        S = P + K_in + c["T"]
        rest = P + T / 2 if c["softmax"] == "causal" else 0
        return dict(bytes=B * (T * q + S * kv + S_out * (kv + 2 * kv + 2 * c["D"] * e + 16 * c["n_pos"])),
                    flops=flops * (K_in + rest) / K_in)
    N, K = c["N"], c["N"] // 4
    return dict(bytes=B * (2 * T * q + K_in * kv + 2 * c["H_q"] * K_in * 4 + 2 * N * 4 + 4 * K), flops=2 * flops)


def tolerance(case):
    # fp32 sums of bf16 or fp32 products: the largest error seen against
    # exact() over these ranges is 1.1e-6 (the fused score, which divides by
    # the MAD); a token that ties with the K-th score moves the kept indices
    # between it and the one it replaces
    return {"rel": 5e-6, "max": 2e-4, "differ": 0.01}


# ----------------------------------------------------------------------------
# the same in float64
# ----------------------------------------------------------------------------


def _exact_prellm(c, seed):
    cls, Z, T, tl = _stage1(c, seed)
    B, N, M = c["B"], c["N"], c["M"]
    seg = cls.double().view(B, c["H_v"], c["n_seg"], N // c["n_seg"])
    sal = torch.softmax(seg, dim=3).view(B, c["H_v"], N).mean(1)
    rel = torch.empty((B, N), device=Z.device, dtype=torch.float64)
    for b in range(B):
        m = M if tl is None else int(tl[b])
        z, t = Z[b].double(), T[b, :m].double()
        z = z / z.norm(dim=1, keepdim=True).clamp_min(1e-12)
        t = t / t.norm(dim=1, keepdim=True).clamp_min(1e-12)
        rel[b] = (z @ t.T).clamp_min(0.0).square().mean(1).sqrt()
    out = dict(idx=None, feats=None, div=None, score=None, sal=sal, rel=rel, norm=None)
    if c["mode"] == "weights":
        norm, branch = [], []
        for s, w, tau in ((sal, 2 * (1 - c["rho"]), 1.4), (rel, 2 * c["rho"], 1.0)):
            med = s.sort(dim=1).values[:, (N - 1) // 2]
            mad = (s - med[:, None]).abs().sort(dim=1).values[:, (N - 1) // 2]
            norm += [med, mad]
            branch.append(w * ((s - med[:, None]) / (mad[:, None] + 1e-8)).clamp_min(0.0) / tau)
        out["score"] = torch.maximum(*branch) + (branch[0] * branch[1]).sqrt()
        out["norm"] = torch.stack(norm, dim=1)
    return out


def _attention(c, q, k, tl, b, softmax):
    """A [H_q, T_b, K_in] of sample b over the visual columns."""
    P, K, G = c["P"], c["K_in"], c["H_q"] // c["H_kv"]
    t = c["T"] if tl is None else int(tl[b])
    keys = k[b].double().repeat_interleave(G, dim=1).permute(1, 2, 0).contiguous()
    rows = q[b, P + K:P + K + t].double().permute(1, 0, 2).contiguous()
    if softmax == "visual":
        return torch.softmax(rows @ keys[:, :, P:P + K].contiguous() * c["d_h"] ** -0.5, dim=2)
    x = rows @ keys[:, :, :P + K + t].contiguous() * c["d_h"] ** -0.5
    later = torch.ones(t, t, device=x.device, dtype=torch.bool).triu(1)
    x[:, :, P + K:].masked_fill_(later, -math.inf)
    return torch.softmax(x, dim=2)[:, :, P:P + K]


def _exact_inllm(c, seed):
    _, _, (q,), k, (tl,) = _stage2(c, seed)
    var, score = [], []
    for b in range(c["B"]):
        A = _attention(c, q, k, tl, b, c["softmax"])
        u = A.var(dim=2, unbiased=False).mean(1)
        heads = u.sort(descending=True, stable=True).indices[:c["n_keep"]]
        var.append(u)
        score.append(A[heads].mean(0).amax(0))
    return dict(idx=None, hidden=None, k=None, v=None, pos=None, heads=None, var=torch.stack(var),
                score=torch.stack(score))


def _exact_analysis(c, seed):
    _, _, qs, k, lens = _stage2(c, seed, questions=2)
    out = dict(ts=None, rho=None, idx=None)
    profiles = []
    for j, (q, tl) in enumerate(zip(qs, lens)):
        p, u = [], []
        for b in range(c["B"]):
            A = _attention(c, q, k, tl, b, "visual")
            p.append(A.mean(1))
            u.append(A.var(dim=2, unbiased=False).mean(1))
        profiles.append(torch.stack(p))
        out["p%d" % j], out["v%d" % j] = profiles[-1], torch.stack(u)
    out["ts"] = 1 - torch.cosine_similarity(profiles[0], profiles[1], dim=2)
    return out


def exact(case, seed):
    f = {"prellm": _exact_prellm, "inllm": _exact_inllm, "analysis": _exact_analysis}[case["kind"]]
    return f(case, seed)
