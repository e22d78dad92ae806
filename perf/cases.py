"""Timed cases of the LM-head log-probability path, through the package's public calls.

Each case is one call (or the few calls that belong together) as a rollout engine
or a trainer makes it: decode batches, packed training micro-batches, the second
reduction order, the backward, the final norm and the per-token statistics. The
listed cases stand for the ranges `draw` samples from. Inputs are synthetic and
made from the seed alone: row-normalised hidden states, N(0, 0.02^2) weights (the
usual initialiser range), tokens drawn from the model's own tempered softmax.
"""

from __future__ import annotations

import math

import torch

import paper_2605_14220_amd as tim
from paper_2605_14220_amd import Estimator, Mode, Order

EPS = 1e-6       # of the final norm
W_STD = 0.02
CHUNK = 2048     # rows per block of the plain torch helpers


def listed():
    return [
        # one scoring step of a toy configuration: norm, head and merge, all launch latency
        {"name": "residual_tiny", "kind": "residual", "T": 64, "d": 256, "V": 4096, "tau": 1.0},
        # a decode step with few responses in flight, outputs preallocated as a serving loop holds them
        {"name": "decode_5", "kind": "decode_noalloc", "T": 5, "d": 2048, "V": 151936, "tau": 1.0},
        # a decode step of 64 responses at temperature 0.7, the widest configuration
        {"name": "decode_64", "kind": "decode", "T": 64, "d": 5120, "V": 152064, "tau": 0.7},
        # a decode step of a fuller, ragged batch
        {"name": "decode_200", "kind": "decode", "T": 200, "d": 4096, "V": 151936, "tau": 1.0},
        # one response scored alone by the trainer, its length no multiple of a tile
        {"name": "train_643", "kind": "train", "T": 643, "d": 4096, "V": 151936, "tau": 1.0, "mb": 0},
        # a packed batch of 16 responses in one call
        {"name": "train_9101", "kind": "train", "T": 9101, "d": 2048, "V": 151936, "tau": 1.0, "mb": 0},
        # a packed stream in micro-batches of 16384 with a ragged last one
        {"name": "train_20011", "kind": "train", "T": 20011, "d": 4096, "V": 151936, "tau": 1.0, "mb": 16384},
        # the same rows by the engine that reduces in another order, for the mismatch between the two
        {"name": "engine2_2048", "kind": "engine2", "T": 2048, "d": 4096, "V": 151936, "tau": 1.0, "mb": 0},
        # gradients of the policy loss over two micro-batches
        {"name": "backward_8000", "kind": "backward", "T": 8000, "d": 4096, "V": 151936, "tau": 1.0, "mb": 4096,
         "entropy": False},
        # gradients of a short batch with an entropy bonus
        {"name": "backward_1001", "kind": "backward", "T": 1001, "d": 2048, "V": 151936, "tau": 1.0, "mb": 0,
         "entropy": True},
        # the final norm of a micro-batch, forward and backward
        {"name": "norm_16384", "kind": "norm", "T": 16384, "d": 4096},
        # token statistics, rejection scores and the clipped loss over a packed stream of 64 responses
        {"name": "losses_64", "kind": "losses", "n": 64, "lo": 512, "hi": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["residual", "decode", "decode_noalloc", "train", "train", "engine2", "backward", "backward",
                       "norm", "losses"])
    if kind == "losses":  # from one short response to many, up to 16384 tokens each
        hi = _log_int(rng, 64, 16384)
        return {"kind": kind, "n": _log_int(rng, 1, min(256, 400000 // hi)), "lo": max(1, hi // 8), "hi": hi}
    if kind == "norm":
        d = rng.choice([256, 1024, 1536, 2048, 3584, 4096, 5120, 8192])
        return {"kind": kind, "T": _log_int(rng, 16, min(140000, 280000000 // d)), "d": d}
    tau = rng.choice([1.0, 1.0, 0.7, 0.6])
    if kind == "residual":
        return {"kind": kind, "T": _log_int(rng, 1, 512), "d": 128 * rng.randint(1, 8), "V": _log_int(rng, 1000, 20000),
                "tau": tau}
    d = rng.choice([1024, 1536, 2048, 3584, 4096, 5120])
    V = rng.choice([32000, 50257, 131072, 151936, 152064])
    case = {"kind": kind, "T": 1, "d": d, "V": V, "tau": tau}
    if kind in ("decode", "decode_noalloc"):
        case["T"] = _log_int(rng, 1, 256)
        return case
    # at most as many tokens as cost the largest listed case of the kind
    top = {"train": 20011 * 4096 * 151936, "engine2": 2048 * 4096 * 151936, "backward": 8000 * 4096 * 151936}[kind]
    case["T"] = _log_int(rng, 65, max(66, min(20011, top // (d * V))))
    case["mb"] = rng.choice([0, 0, 4096, 16384])
    if kind == "backward":
        case["entropy"] = rng.random() < 0.5
    return case


def _gen(seed, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 16 + k)
    return g


def _hidden(T, d, g):
    x = torch.randn((T, d), generator=g, dtype=torch.float32, device="cuda")
    return (x * torch.rsqrt(x.square().mean(dim=1, keepdim=True) + EPS)).to(torch.bfloat16)


def _weights(V, d, g):
    w = torch.empty((V, d), dtype=torch.bfloat16, device="cuda")
    for r in range(0, V, 16384):
        n = min(16384, V - r)
        w[r:r + n] = (torch.randn((n, d), generator=g, dtype=torch.float32, device="cuda") * W_STD).to(torch.bfloat16)
    return w


def _tokens(h, w, tau, g):
    """Tokens drawn from softmax(h w^T / tau): the largest of p / Exp(1)."""
    out = torch.empty(h.shape[0], dtype=torch.int32, device="cuda")
    for r in range(0, h.shape[0], CHUNK):
        p = torch.softmax((h[r:r + CHUNK] @ w.T).float() / tau, dim=1)
        e = torch.empty_like(p).exponential_(generator=g).clamp_(min=1e-30)
        out[r:r + CHUNK] = torch.argmax(p / e, dim=1).to(torch.int32)
    return out


def _head64(h, w, tokens, tau, each=None):
    """(logp, entropy, lse) in float64; each(row0, z - lse, entropy) sees every block of rows."""
    w64 = w.double()
    T = h.shape[0]
    lp, ent, lse = (torch.empty(T, dtype=torch.float64, device=h.device) for _ in range(3))
    for r in range(0, T, CHUNK):
        z = (h[r:r + CHUNK].double() @ w64.T) / tau
        s = slice(r, r + z.shape[0])
        lse[s] = torch.logsumexp(z, dim=1)
        q = z.sub_(lse[s, None])
        lp[s] = q.gather(1, tokens[s].long()[:, None])[:, 0]
        ent[s] = -(torch.exp(q) * q).sum(dim=1)
        if each is not None:
            each(r, q, ent[s], w64)
    return lp, ent, lse


def _lengths(case, seed):
    """The case's response lengths, uniform in [lo, hi], in the seed's order (one token count for all seeds)."""
    lens = torch.randint(case["lo"], case["hi"] + 1, (case["n"],), generator=torch.Generator().manual_seed(case["hi"]))
    return lens[torch.randperm(case["n"], generator=torch.Generator().manual_seed(int(seed)))]


def prepare(case, seed):
    kind = case["kind"]
    g = [_gen(seed, k) for k in range(6)]
    st = {"kind": kind}
    if kind == "losses":  # log-probs of a rollout engine and of a trainer: tiny
        # discrepancies everywhere, a heavy tail on 1% of the tokens of about half of the responses (those are rejected)
        lens = _lengths(case, seed)
        cu = torch.zeros(case["n"] + 1, dtype=torch.int64)
        cu[1:] = torch.cumsum(lens, 0)
        T = int(cu[-1])
        st["cu"] = cu.cuda()
        b = -2.0 * torch.empty(T, device="cuda").exponential_(generator=g[0])
        torn = torch.repeat_interleave(torch.rand(case["n"], device="cuda", generator=g[5]) < 0.5, lens.cuda())
        tail = (torch.rand(T, device="cuda", generator=g[1]) < 0.01) & torn
        a = b + torch.randn(T, device="cuda", generator=g[2]) * torch.where(tail, 0.3, 1e-5)
        old = a + 0.1 * torch.randn(T, device="cuda", generator=g[3])  # the policy a few updates back
        st["train"], st["rollout"], st["old"] = a, b, old
        adv = torch.randn(case["n"], device="cuda", generator=g[4])
        st["adv"] = torch.repeat_interleave(adv, lens.cuda())
        return st
    T, d = case["T"], case["d"]
    if kind in ("norm", "residual"):
        st["x"] = (2.0 * torch.randn((T, d), device="cuda", generator=g[0])).to(torch.bfloat16)
        st["gamma"] = (1.0 + 0.1 * torch.randn(d, device="cuda", generator=g[3])).to(torch.bfloat16)
    if kind == "norm":
        st["grad_h"] = 1e-3 * torch.randn((T, d), device="cuda", generator=g[4])
        return st
    st["tau"] = case["tau"]
    st["w"] = _weights(case["V"], d, g[1])
    if kind == "residual":
        n = st["x"].float()
        h = (n * torch.rsqrt(n.square().mean(dim=1, keepdim=True) + EPS)).to(torch.bfloat16) * st["gamma"]
    else:
        h = st["h"] = _hidden(T, d, g[0])
    st["tokens"] = _tokens(h, st["w"], case["tau"], g[2])
    st["mb"] = case.get("mb", 0)
    if kind == "decode_noalloc":
        st["out"] = tuple(torch.empty(T, dtype=torch.float32, device="cuda") for _ in range(2)) + (None,)
    if kind == "backward":  # what the forward and the loss left behind
        _, ent, lse = _head64(h, st["w"], st["tokens"], case["tau"])
        st["lse"], st["ent"] = lse.float(), ent.float()
        st["g"] = torch.randn(T, device="cuda", generator=g[4])
        st["e"] = torch.full((T,), 0.1, device="cuda") if case["entropy"] else None
        need = tim.backward_workspace_size(T, d, case["V"], case["mb"])
        st["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    return st


def run(st):
    kind = st["kind"]
    if kind == "residual":
        return tim.logprobs_from_residual(st["x"], st["gamma"], st["w"], st["tokens"], EPS, st["tau"], lse=True)
    if kind == "decode":
        return tim.logprobs(st["h"], st["w"], st["tokens"], st["tau"], mode=Mode.ROLLOUT)[:2]
    if kind == "decode_noalloc":
        return tim.logprobs_noalloc(st["h"], st["w"], st["tokens"], st["tau"], mode=Mode.ROLLOUT, out=st["out"])[:2]
    if kind == "train":
        return tim.logprobs(st["h"], st["w"], st["tokens"], st["tau"], micro_batch=st["mb"], lse=True)
    if kind == "engine2":
        return tim.logprobs(st["h"], st["w"], st["tokens"], st["tau"], micro_batch=st["mb"], order=Order.SPLITK4)[:2]
    if kind == "backward":
        ent = st["ent"] if st["e"] is not None else None
        return tim.logprobs_backward(st["h"], st["w"], st["tokens"], st["lse"], st["g"], st["tau"], entropy=ent,
                                     grad_entropy=st["e"], micro_batch=st["mb"], workspace=st["ws"])
    if kind == "norm":
        h, rstd = tim.rmsnorm(st["x"], st["gamma"], EPS)
        gx, gg = tim.rmsnorm_backward(st["x"], st["gamma"], rstd, st["grad_h"])
        return h, rstd, gx, gg
    stats = tim.mismatch(st["train"], st["rollout"])
    score, keep, weight = tim.mismatch_seq(st["train"], st["rollout"], st["cu"], estimator=Estimator.K3)
    loss = tim.ppo_loss(st["train"], st["old"], st["adv"], st["cu"], weight=weight)
    return (*stats, score, keep, weight, loss)


def work(case):
    """Bytes of the inputs read once and the outputs written once, and the contractions' operations."""
    kind = case["kind"]
    if kind == "losses":
        T = case["n"] * (case["lo"] + case["hi"]) // 2
        # logp, rollout logp, old logp and advantage in; 4 statistics, loss, gradient, contribution, mask out
        return {"bytes": T * (16 + 16 + 13) + case["n"] * (8 + 8 + 1 + 8), "flops": 60 * T}
    T, d = case["T"], case["d"]
    if kind == "norm":  # x, grad_h in; h, grad_x out
        return {"bytes": T * d * (2 + 4 + 2 + 4) + 4 * T + 6 * d, "flops": 14 * T * d}
    V = case["V"]
    if kind == "backward":
        return {"bytes": 2 * T * d + 2 * V * d + 4 * T * d + 4 * V * d + 16 * T, "flops": 6 * T * d * V}
    b = 2 * T * d + 2 * V * d + 16 * T
    if kind == "residual":
        b += 2 * T * d
    return {"bytes": b, "flops": 2 * T * d * V}


def tolerance(case):
    return TOLERANCE[case["kind"]]


# About four times what the path shows against `exact` over the ranges above (logp 2e-7, gradients 1.7e-3: the
# logit gradients' rounding to bf16; norm 2.3e-5: values that straddle a bf16 rounding boundary, a code apart).
TOLERANCE = {
    "residual": {"rel": 1e-4, "max": 1.6e-2},
    "decode": {"rel": 1e-6},
    "decode_noalloc": {"rel": 1e-6},
    "train": {"rel": 1e-6},
    "engine2": {"rel": 1e-6},
    "backward": {"rel": 7e-3},
    "norm": {"rel": 1e-4, "max": 1.6e-2},
    "losses": {"rel": 4e-7, "differ": 0.0},
}


def _norm64(x, gamma):
    """The norm in float64 with its two roundings to bf16: (h, rstd, x in float64)."""
    x64 = x.double()
    r = 1.0 / torch.sqrt(x64.square().mean(dim=1) + EPS)
    n = (x64 * r[:, None]).to(torch.bfloat16).double()
    return (n * gamma.double()).to(torch.bfloat16).double(), r, x64


def exact(case, seed):
    kind = case["kind"]
    st = prepare(case, seed)
    if kind == "losses":
        return _losses64(st)
    if kind == "norm":
        h, r, x = _norm64(st["x"], st["gamma"])
        gg = st["grad_h"].double() * st["gamma"].double()
        s = (gg * x).sum(dim=1, keepdim=True)
        gx = r[:, None] * gg - (r[:, None] ** 3 / case["d"]) * s * x
        return h, r, gx, (st["grad_h"].double() * x * r[:, None]).sum(dim=0)
    if kind == "residual":
        h, r, _ = _norm64(st["x"], st["gamma"])
        lp, ent, lse = _head64(h, st["w"], st["tokens"], case["tau"])
        return lp, ent, lse, h, r
    if kind == "backward":
        gh = torch.empty(st["h"].shape, dtype=torch.float64, device="cuda")
        gw = torch.zeros(st["w"].shape, dtype=torch.float64, device="cuda")

        def grads(r0, q, ent, w64):
            s = slice(r0, r0 + q.shape[0])
            p = torch.exp(q)
            dz = -st["g"][s, None].double() * p
            if st["e"] is not None:
                dz -= st["e"][s, None].double() * p * (q + ent[:, None])
            dz.scatter_add_(1, st["tokens"][s].long()[:, None], st["g"][s, None].double())
            dz /= case["tau"]
            gh[s] = dz @ w64
            gw.addmm_(dz.T, st["h"][s].double())

        _head64(st["h"], st["w"], st["tokens"], case["tau"], grads)
        return gh, gw
    lp, ent, lse = _head64(st["h"], st["w"], st["tokens"], case["tau"])
    return (lp, ent, lse) if kind == "train" else (lp, ent)


def _losses64(st):
    a, b = st["train"].double(), st["rollout"].double()
    cu = st["cu"]
    n = cu.numel() - 1
    seg = torch.repeat_interleave(torch.arange(n, device=cu.device), cu[1:] - cu[:-1])

    def per_response(v):
        return torch.zeros(n, dtype=torch.float64, device=v.device).index_add_(0, seg, v)

    d = a - b
    series = sum(d ** k / math.factorial(k) for k in range(2, 10))
    k3 = torch.where(d.abs() < 2.0 ** -5, series, torch.expm1(d) - d)
    w = torch.exp(d).clamp(max=2.0)
    score = per_response(k3)
    keep = score <= 1e-3
    weight = torch.where(keep[seg], w, torch.zeros_like(w))
    dl = a - st["old"].double()
    adv = st["adv"].double()
    w32 = weight.float().double()  # the loss takes the weights as the call before it returns them
    r = torch.exp(dl)
    lo, hi = 1.0 - float(torch.tensor(0.2, dtype=torch.float32)), 1.0 + float(torch.tensor(0.2, dtype=torch.float32))
    clip = ((adv > 0) & (dl > math.log(hi))) | ((adv < 0) & (dl < math.log(lo)))
    tl = w32 * torch.where(clip, -adv * torch.where(adv > 0, hi, lo), -adv * r)
    seq = per_response(tl)
    loss = {"seq_loss": seq, "batch_loss": seq.mean().reshape(1), "token_loss": tl,
            "grad": torch.where(clip, torch.zeros_like(r), -w32 * adv * r / n), "contribution": -(r - 1.0) * adv,
            "clipped": clip.to(torch.uint8)}
    return d, k3, w, score, keep.to(torch.uint8), weight, loss
