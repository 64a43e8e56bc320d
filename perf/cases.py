"""What a program that trains a vision-language-action policy has this library do, as measurable cases.

One update of such a program: roll out parallel environments (prefill the observation prefix, decode the action
tokens one after the other or as one parallel chunk), turn rewards into advantages and the clipped objective,
recompute the log-probabilities of the stored actions, and take the LoRA gradients.  The decoder is the 7B shape
(hidden 4096, 32 heads, FFN 11008, bf16) or the tiny fp32 one.  Every layer of a decoder does the same work, so the cases
run a few layers of the 7B shape (0.4 GB of weights each, far more than any cache holds).

Weights are N(0, 0.02), patch embeddings N(0, 1), norm gains 1 + N(0, 0.02), LoRA factors N(0, 0.05).  Autoregressive
bf16 decodes draw each token's Gumbel noise with one bin raised far above the rest: the tokens then replay a
drawn action sequence, which two correct implementations agree on, and the logits of all tokens are comparable.
The parallel chunk and the fp32 decoder sample with plain Gumbel noise.
"""
import math
from types import SimpleNamespace

import torch

from paper_2510_06710_amd import binding as vb
from paper_2510_06710_amd.harness import Rollout

DEV = "cuda:0"
SHAPES = {
    "7b": dict(hidden=4096, n_heads=32, ffn=11008, vocab=32000, dtype="bf16"),
    "tiny": dict(hidden=256, n_heads=4, ffn=688, vocab=1024, dtype="f32"),
}
RMS_EPS, ROPE_THETA, N_BINS = 1e-5, 10000.0, 256
VALUE_DIM, VALUE_BIAS = 8, 0.25     # one value per action of an 8-step chunk
GAMMA, LAMBDA, CLIP_LOW, CLIP_HIGH, GROUP = 0.99, 0.95, 0.2, 0.28, 8
PROJ = ("q", "k", "v", "o", "gate", "up", "down")


def listed():
    return [
        # the tiny fp32 decoder, 8 environments: a unit test or a toy run, all launches and latency
        dict(name="rollout_tiny_f32", kind="rollout", shape="tiny", layers=2, batch=8, patches=48, instr=16, tokens=7, temp=1.0),
        # one robot waiting for its next action: every weight read once a forward
        dict(name="rollout_b1", kind="rollout", shape="7b", layers=8, batch=1, patches=256, instr=32, tokens=7, temp=1.0),
        # a handful of environments with an instruction length that is no multiple of anything, sampled at 1.6
        dict(name="rollout_b13_odd", kind="rollout", shape="7b", layers=4, batch=13, patches=243, instr=18, tokens=7, temp=1.6),
        # one simulator step of 64 environments
        dict(name="rollout_b64", kind="rollout", shape="7b", layers=4, batch=64, patches=256, instr=32, tokens=7, temp=1.0),
        # the observation prefix of 256 environments, the largest pass of a rollout, with its KV cache
        dict(name="prefill_b256", kind="prefill", shape="7b", layers=4, batch=256, patches=256, instr=32, tokens=7, temp=1.0),
        # the seven action tokens of 256 environments against that cache
        dict(name="decode_b256", kind="decode", shape="7b", layers=4, batch=256, patches=256, instr=32, tokens=7, temp=1.0),
        # parallel chunk of 8 actions x 7 dimensions for 128 environments
        dict(name="chunk_b128", kind="chunk", shape="7b", layers=4, batch=128, patches=256, instr=32, tokens=56, temp=1.0),
        # chunk of 25 actions for three evaluation environments
        dict(name="chunk_b3_a175", kind="chunk", shape="7b", layers=4, batch=3, patches=256, instr=25, tokens=175, temp=1.6),
        # log-prob recompute of 80 stored rollouts in micro-batches of 40
        dict(name="recompute_n80", kind="recompute", shape="7b", layers=4, batch=80, micro=40, patches=256, instr=32, tokens=7, temp=1.0),
        # LoRA gradients of one micro-batch of 32 rollouts, layers run a second time
        dict(name="backward_n32_r32", kind="backward", shape="7b", layers=2, batch=32, micro=32, patches=256, instr=32, tokens=7, temp=1.0,
             rank=32, keep=False),
        # the same for a short micro-batch at rank 8 with every activation kept
        dict(name="backward_keep_n7_r8", kind="backward", shape="7b", layers=2, batch=7, micro=7, patches=256, instr=21, tokens=7, temp=1.0,
             rank=8, keep=True),
        # advantages and objective of an epoch: 256 environments x 80 steps, groups of 8
        dict(name="objective_256x80", kind="objective", traj=256, steps=80),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rollout", "rollout", "tiny", "prefill", "decode", "chunk", "recompute", "backward", "objective"])
    if kind == "objective":
        return dict(kind=kind, traj=GROUP * _log(rng, 1, 64), steps=_log(rng, 3, 512))
    c = dict(kind=kind, shape="7b", layers=4, patches=rng.randint(64, 256), instr=rng.randint(4, 40), tokens=rng.randint(4, 8),
             temp=rng.choice([1.0, 1.6]))
    if kind == "tiny":
        return dict(c, kind="rollout", shape="tiny", layers=2, batch=_log(rng, 1, 64), patches=rng.randint(8, 64))
    if kind == "rollout":
        return dict(c, batch=_log(rng, 1, 64))
    if kind in ("prefill", "decode"):
        return dict(c, batch=_log(rng, 1, 256))
    if kind == "chunk":
        a = 7 * rng.randint(2, 25)
        return dict(c, tokens=a, batch=_log(rng, 1, 7168 // a))
    if kind == "recompute":
        return dict(c, batch=_log(rng, 1, 80), micro=rng.choice([32, 40]))
    n = _log(rng, 1, 32)
    return dict(c, layers=2, batch=n, micro=n, rank=rng.choice([4, 8, 16, 32]), keep=rng.choice([False, True]))


# ------------------------------------------------------------------------------------------------ inputs
class _Model:
    """A decoder with random weights, in the form that the harness takes."""

    def __init__(self, case, gen):
        self.device, self.gen = DEV, gen
        self.shape = SimpleNamespace(**SHAPES[case["shape"]], n_layers=case["layers"], n_bins=N_BINS, rms_eps=RMS_EPS, rope_theta=ROPE_THETA)
        for k, v in vars(self.shape).items():
            setattr(self, k, v)
        self.torch_dtype = torch.float32 if self.dtype == "f32" else torch.bfloat16
        H, F = self.hidden, self.ffn
        sizes = dict(attn_norm=(H,), wq=(H, H), wk=(H, H), wv=(H, H), wo=(H, H), ffn_norm=(H,), w_gate=(F, H), w_up=(F, H), w_down=(H, F))
        self.layers = [{n: self._gain() if len(z) == 1 else self._mat(*z) for n, z in sizes.items()} for _ in range(self.n_layers)]
        self._embed, self._head = self._mat(self.vocab, H), self._mat(self.vocab, H)
        self._final, self._vw = self._gain(), 0.02 * torch.randn(VALUE_DIM, H, device=DEV, generator=gen)
        self._vb = torch.randn(VALUE_DIM, device=DEV, generator=gen)

    def _mat(self, *size):
        return torch.empty(*size, dtype=self.torch_dtype, device=DEV).normal_(0.0, 0.02, generator=self.gen)

    def _gain(self):
        return 1.0 + 0.02 * torch.randn(self.hidden, device=DEV, generator=self.gen)

    layer = lambda self, l: self.layers[l]  # noqa: E731
    embed = lambda self: self._embed  # noqa: E731
    lm_head = lambda self: self._head  # noqa: E731
    final_norm = lambda self: self._final  # noqa: E731
    value_w = lambda self, dim: self._vw  # noqa: E731
    value_bias = lambda self, dim: self._vb  # noqa: E731


def _inputs(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    if case["kind"] == "objective":
        n, t = case["traj"], case["steps"]
        old = -3.0 * torch.randn(n, t, device=DEV, generator=g).abs()
        return dict(
            rewards=torch.randn(n, t, device=DEV, generator=g), values=torch.randn(n, t + 1, device=DEV, generator=g),
            dones=(torch.rand(n, t, device=DEV, generator=g) < 0.02).int(), total=(torch.rand(n, device=DEV, generator=g) < 0.5).float(),
            old=old, new=old + 0.25 * torch.randn(n, t, device=DEV, generator=g),
            mask=(torch.arange(t, device=DEV)[None, :] < torch.randint(0, t + 1, (n, 1), device=DEV, generator=g)).int().contiguous())
    m = _Model(case, g)
    B, P, T, A, H = case["batch"], case["patches"], case["instr"], case["tokens"], m.hidden
    d = dict(model=m, patch=torch.randn(B, P, H, device=DEV, generator=g).to(m.torch_dtype),
             ids=torch.randint(0, m.vocab - N_BINS, (B, T), device=DEV, generator=g, dtype=torch.int32),
             bins=torch.randint(0, N_BINS, (B, A), device=DEV, generator=g, dtype=torch.int32), slot=None)
    if case["kind"] == "chunk":
        d["slot"] = m._mat(A, H)
    if case["kind"] in ("rollout", "decode", "chunk"):
        u = torch.rand(B, A, N_BINS, device=DEV, generator=g, dtype=torch.float64).clamp_(2.0 ** -25, 1.0 - 2.0 ** -25)
        d["gumbel"] = -(-u.log()).log()
        if case["kind"] != "chunk" and m.dtype == "bf16":
            d["gumbel"].scatter_add_(2, d["bins"].long()[..., None], torch.full((B, A, 1), 64.0, dtype=torch.float64, device=DEV))
        d["gumbel"] = d["gumbel"].float()
    if case["kind"] == "backward":
        r, dims = case["rank"], {p: (H, H) for p in "qkvo"} | dict(gate=(m.ffn, H), up=(m.ffn, H), down=(H, m.ffn))
        rand = lambda *z: (0.05 * torch.randn(*z, device=DEV, generator=g)).to(m.torch_dtype)  # noqa: E731
        d["lora"] = [{p: (rand(r, i), rand(o, r)) for p, (o, i) in dims.items()} for _ in range(m.n_layers)]
        d["coef"] = torch.randn(B, A, device=DEV, generator=g)
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    state = dict(case=case, **d)
    if case["kind"] == "objective":
        return state
    S = case["patches"] + case["instr"]
    run = Rollout(d["model"], case.get("micro", case["batch"]), S + case["tokens"], device=DEV, value_b=VALUE_BIAS, value_dim=VALUE_DIM)
    state["run"], state["S"] = run, S
    if case["kind"] not in ("recompute", "backward"):
        state["kv"] = run.kv(case["batch"], S + case["tokens"]).zero_().view(d["model"].torch_dtype)
    if case["kind"] in ("decode", "chunk"):
        state["h_last"] = run.prefill(d["patch"], d["ids"])[0]
    return state


# ------------------------------------------------------------------------------------------------ the calls
def run(state):
    c, kind = state["case"], state["case"]["kind"]
    if kind == "objective":
        return _run_objective(state)
    r, S, A, t = state["run"], state["S"], c["tokens"], c["temp"]
    if kind == "rollout":
        h, value = r.prefill(state["patch"], state["ids"])
        bins, logp, ent, logits = r.decode(h, S, A, 0, None, t, state["gumbel"])
        return dict(h_last=h, value=value, bins=bins, logp=logp, entropy=ent, logits=logits, kv=state["kv"])
    if kind == "prefill":
        h, value = r.prefill(state["patch"], state["ids"])
        return dict(h_last=h, value=value, kv=state["kv"])
    if kind in ("decode", "chunk"):
        bins, logp, ent, logits = r.decode(state["h_last"], S, A, int(kind == "chunk"), state["slot"], t, state["gumbel"])
        return dict(bins=bins, logp=logp, entropy=ent, logits=logits, kv=state["kv"])
    if kind == "recompute":
        logp, ent, value, logits = r.recompute(state["patch"], state["ids"], state["bins"], A, 0, None, t)
        return dict(logp=logp, entropy=ent, value=value, logits=logits)
    grads, logp = r.backward(state["patch"], state["ids"], state["bins"], state["coef"], A, state["lora"], c["rank"], 0.5, 0, None, t,
                             keep_activations=c["keep"])
    return dict(logp=logp, grads=[{p: list(layer[p]) for p in PROJ} for layer in grads])


def _run_objective(s):
    n, t = s["case"]["traj"], s["case"]["steps"]
    new = lambda *z, dtype=torch.float32: torch.empty(*z, dtype=dtype, device=DEV)  # noqa: E731
    adv, returns, gadv, keep = new(n, t), new(n, t), new(n), new(n // GROUP, dtype=torch.int32)
    vb.vla_gae(s["rewards"], s["values"], s["dones"], n, t, GAMMA, LAMBDA, adv, returns)
    vb.vla_grpo_advantage(s["total"], n // GROUP, GROUP, gadv, keep)
    ws = new(vb.vla_policy_objective_workspace_bytes(n), dtype=torch.uint8)
    out = dict(adv=adv, returns=returns, gadv=gadv, keep=keep)
    for name, a, per_step in (("ppo", adv, True), ("grpo", gadv, False)):
        obj, per, frac = new(1), new(n, t), new(1)
        vb.vla_policy_objective(s["new"], s["old"], a, per_step, s["mask"], n, t, CLIP_LOW, CLIP_HIGH, not per_step, ws, obj, per, frac)
        out[name] = [obj, per, frac]
    return out


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    if case["kind"] == "objective":
        n, t = case["traj"], case["steps"]
        # rewards, values, dones, new, old, mask in; advantages, returns, two masked surrogates out
        return {"bytes": 4.0 * (10 * n * t + 4 * n), "flops": 40.0 * n * t}
    s = SHAPES[case["shape"]]
    H, F, es = s["hidden"], s["ffn"], 4 if s["dtype"] == "f32" else 2
    L, B, A, S, kind = case["layers"], case["batch"], case["tokens"], case["patches"] + case["instr"], case["kind"]
    params, kv_row = 4 * H * H + 3 * H * F, 2 * H * es
    weights = L * params * es

    def rows_flops(rows, keys, tail):
        """`rows` per sequence over `keys` visible (query, key) pairs; the last layer's output is needed for `tail` rows only."""
        full = 2.0 * rows * params + 4.0 * H * keys
        last = 2.0 * rows * 2 * H * H + 2.0 * tail * (params - 2 * H * H) + 4.0 * H * keys * tail / rows
        return B * ((L - 1) * full + last)

    def causal(r):
        return r * (r + 1) / 2.0

    head = 2.0 * B * A * N_BINS * H
    obs = B * case["patches"] * H * es + B * H * 4
    b = f = 0.0
    if kind in ("rollout", "prefill"):
        f += rows_flops(S, causal(S), 1)
        b += weights + obs + L * B * S * kv_row
    if kind in ("rollout", "decode"):
        f += head + B * L * sum(2.0 * params + 4.0 * H * (S + j + 1) for j in range(A - 1))
        b += (A - 1) * weights + A * N_BINS * H * es + B * A * N_BINS * 8 + L * B * kv_row * sum(S + j + 1 for j in range(A - 1))
    if kind == "chunk":
        f += head + B * L * A * (2.0 * params + 4.0 * H * (S + A))
        b += weights + N_BINS * H * es + B * A * N_BINS * 8 + L * B * kv_row * (S + 2 * A)
    if kind in ("recompute", "backward"):
        f += head + rows_flops(S + A - 1, causal(S + A - 1), A)
        b += weights + obs + N_BINS * H * es + B * A * N_BINS * 4
    if kind == "backward":
        factors = L * case["rank"] * (8 * H + 3 * (H + F))
        f += head + rows_flops(S + A - 1, 2 * causal(S + A - 1), A) + 8.0 * B * (S + A - 1) * factors
        b += factors * (es + 4)
    return {"bytes": b, "flops": f}


def tolerance(case):
    if case["kind"] == "objective" or SHAPES[case["shape"]]["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}   # against 64 bits: 1e-6 at most
    # against 64 bits: 1.5e-2 after 4 layers, whose operands are rounded to bf16; chunk bins differ at near ties
    return {"rel": 3e-2, "max": 0.5, "differ": 0.01}


# ------------------------------------------------------------------------------------------------ the same in 64 bits
def _norm(x, gain):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + RMS_EPS) * gain.double()


def _rotate(x, pos):
    """x [n, rows, heads, d], half-split pairing."""
    d = x.shape[-1]
    ang = pos.double()[:, None] * ROPE_THETA ** (-torch.arange(0, d, 2, device=DEV, dtype=torch.float64) / d)
    co, si = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., : d // 2], x[..., d // 2:]
    return torch.cat((a * co - b * si, b * co + a * si), -1)


def _lora_product(x, w, factors, proj):
    y = x @ w.double().T
    if factors is not None:
        a, b = factors[proj]
        extra = 0.5 * (x.detach() @ a.T) @ b.T
        y = y + extra - extra.detach()      # value and input gradient of the effective weight, gradients of the factors
    return y


def _hidden(m, x, visible, lora=None):
    """Final-norm output of every row; x [n, rows, hidden]."""
    n, R, H = x.shape
    nh = m.n_heads
    d, pos = H // nh, torch.arange(R, device=DEV)
    for l in range(m.n_layers):
        w, f = m.layer(l), None if lora is None else lora[l]
        z = _norm(x, w["attn_norm"])
        q, k, v = (_lora_product(z, w["w" + p], f, p).view(n, R, nh, d) for p in "qkv")
        q, k, v = _rotate(q, pos).transpose(1, 2), _rotate(k, pos).transpose(1, 2), v.transpose(1, 2)
        p = ((q @ k.transpose(2, 3)) / math.sqrt(d)).masked_fill(~visible, -math.inf).softmax(-1)
        x = x + _lora_product((p @ v).transpose(1, 2).reshape(n, R, H), w["wo"], f, "o")
        z = _norm(x, w["ffn_norm"])
        g = _lora_product(z, w["w_gate"], f, "gate")
        x = x + _lora_product(g * g.sigmoid() * _lora_product(z, w["w_up"], f, "up"), w["w_down"], f, "down")
    return _norm(x, m.final_norm())


def _stats(logits, bins, temp):
    lp = (logits / temp).log_softmax(-1)
    return lp.gather(-1, bins.long()[..., None])[..., 0], -(lp.exp() * lp).sum(-1)


def _exact_rows(case, d, lora=None):
    """(final-norm output of the last prefix row [B, H], logits [B, A, 256]) with the drawn bins as the action tokens."""
    m, S, A = d["model"], case["patches"] + case["instr"], case["tokens"]
    chunk, sampled = case["kind"] == "chunk", case["kind"] == "rollout" and m.dtype == "f32"
    R = S + (A if chunk else A - 1)
    vis = torch.ones(R, R, dtype=torch.bool, device=DEV).tril_()
    if chunk:
        vis[S:] = True
    head, embed = m.lm_head()[m.vocab - N_BINS:].double(), m.embed()
    hs, zs, step = [], [], max(1, 9216 // R) if lora is None else case["batch"]
    for i in range(0, case["batch"], step):
        part = slice(i, i + step)
        prefix = torch.cat((d["patch"][part].double(), embed[d["ids"][part].long()].double()), 1)
        bins = d["bins"][part].long()
        for j in range(A if sampled else 1):
            tail = d["slot"].double()[None].expand(len(bins), -1, -1) if chunk else embed[m.vocab - N_BINS + bins[:, : A - 1]].double()
            h = _hidden(m, torch.cat((prefix, tail), 1), vis, lora)
            z = h[:, S if chunk else S - 1:] @ head.T
            if sampled:                     # token j follows from the tokens before it
                bins[:, j] = (z[:, j] / case["temp"] + d["gumbel"][part][:, j].double()).argmax(-1)
        if sampled:
            d["bins"][part] = bins.int()
        hs.append(h[:, S - 1]), zs.append(z)
    return torch.cat(hs), torch.cat(zs)


def exact(case, seed):
    d = _inputs(case, seed)
    if case["kind"] == "objective":
        return _exact_objective(case, d)
    m = d["model"]
    if case["kind"] == "backward":
        lora = [{p: tuple(t.double().requires_grad_() for t in layer[p]) for p in PROJ} for layer in d["lora"]]
        z = _exact_rows(case, d, lora)[1]
        logp = _stats(z, d["bins"], case["temp"])[0]
        (logp * d["coef"].double()).sum().backward()
        return dict(logp=logp.detach(), grads=[{p: [t.grad for t in layer[p]] for p in PROJ} for layer in lora])
    h, z = _exact_rows(case, d)
    bins = d["bins"]
    if case["kind"] == "chunk":
        bins = (z / case["temp"] + d["gumbel"].double()).argmax(-1)
    value = h @ m.value_w(VALUE_DIM).double().T + VALUE_BIAS + m.value_bias(VALUE_DIM).double()
    logp, ent = _stats(z, bins, case["temp"])
    if case["batch"] * min(case["tokens"], VALUE_DIM) < 50:
        # a handful of numbers: the norm of their errors is a matter of luck, and h_last and the logits show the same errors
        value = logp = ent = None
    if case["kind"] == "prefill":
        return dict(h_last=h, value=value, kv=None)
    if case["kind"] == "chunk":             # a sampled bin may be another one at a near tie, and its log-probability with it
        return dict(bins=None, logp=None, entropy=ent, logits=z, kv=None)
    if case["kind"] == "recompute":
        return dict(logp=logp, entropy=ent, value=value, logits=z)
    out = dict(bins=None, logp=logp, entropy=ent, logits=z, kv=None)
    return dict(out, h_last=h, value=value) if case["kind"] == "rollout" else out


def _exact_objective(case, d):
    n, t = case["traj"], case["steps"]
    r, v, live, total = d["rewards"].double(), d["values"].double(), 1.0 - d["dones"].double(), d["total"].double()
    adv, run_ = torch.zeros(n, t, dtype=torch.float64, device=DEV), torch.zeros(n, dtype=torch.float64, device=DEV)
    for k in reversed(range(t)):
        run_ = r[:, k] + GAMMA * v[:, k + 1] * live[:, k] - v[:, k] + GAMMA * LAMBDA * live[:, k] * run_
        adv[:, k] = run_
    g = total.view(-1, GROUP)
    std = g.std(1, unbiased=False, keepdim=True)
    gadv = torch.where(std > 0, (g - g.mean(1, keepdim=True)) / std.clamp_min(1e-300), torch.zeros_like(g)).reshape(-1)
    out = dict(adv=adv, returns=adv + v[:, :t], gadv=gadv, keep=None)
    rho, mask = (d["new"].double() - d["old"].double()).exp(), d["mask"].double()
    for name, a, per_step in (("ppo", adv, True), ("grpo", gadv[:, None], False)):
        free, cut = rho * a, rho.clamp(1.0 - CLIP_LOW, 1.0 + CLIP_HIGH) * a
        s = torch.minimum(free, cut) * mask
        per_traj = s.sum(1) / mask.sum(1).clamp_min(1.0)
        obj = s.sum() / mask.sum() if per_step else per_traj.mean()
        out[name] = [obj[None], s, (((cut < free) * mask).sum() / mask.sum())[None]]
    return out
