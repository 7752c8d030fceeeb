"""The work a user has the DPPO library do, as cases that can be timed and compared.

A case is a dict of plain values; `path` names the public entry points one pass goes through:

  step         the whole policy update on one batch of rollouts: dppo_select -> dppo_pack ->
               dppo_gather_f32 (advantages, weights) -> dppo_loss_fwd_bwd
  loss         dppo_loss_fwd_bwd alone on packed sequences that are at hand (one micro-batch of an
               update that accumulates gradients, or an update that packs ahead of time)
  logprob      dppo_token_logprob: old-policy / reference log-probs of finished completions
  noalloc      dppo_token_logprob_noalloc: the same from a serving loop that may not allocate
  select_pack  what happens to a batch of rollouts before the model runs: selection, carry-forward
               scores, token-normalised weights, packing, and the two gathers
  prompts      packing a whole prompt dataset before any rollout

Lengths, rewards and pruning uniforms of a case follow from its `rollout` number, so the sizes of
all arrays belong to the case; token ids, hidden states, the vocabulary matrix, the behaviour and
reference log-probs and the arrival order come from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2603_04135_amd as P

DEV = "cuda:0"
CLIP, BETA, NOISE = 0.2, 0.04, 0.05
# Prompt and completion length mixes: (prompt range, completion law)
MIXES = {
    "tiny": ((8, 16), ("uniform", 8, 32)),
    "small": ((64, 256), ("uniform", 128, 1024)),
    "math": ((64, 512), ("lognormal", 1200.0, 0.6, 16, 4096)),
    "long_math": ((64, 512), ("lognormal", 2000.0, 0.6, 16, 8192)),
    "bimodal": ((16, 2048), ("bimodal", 16, 128, 4096, 16384)),
    "short": ((16, 256), ("uniform", 16, 128)),
}


def listed():
    small = dict(D=1024, V=32000, mix="small", r_q=0.4, r_o=0.5, capacity=4096, n_win=32)
    q4b = dict(dtype="bf16", D=2560, V=151936, mix="math")
    q8b = dict(dtype="bf16", D=4096, V=151936)
    return [
        # the smallest batch anyone runs (unit tests, debugging a training script): all latency and launches
        dict(name="tiny_step_f32", path="step", dtype="f32", D=64, V=512, Q=4, G=4, mix="tiny", r_q=0.5, r_o=0.5,
             capacity=256, n_win=4, rollout=1),
        # a small model's whole update: short contraction, small vocabulary
        dict(small, name="small_step", path="step", dtype="bf16", Q=32, G=8, rollout=2),
        # the headline: one whole update of a Qwen3-4B-shaped policy, 64 prompts x 8 completions
        dict(q4b, name="qwen3_4b_step", path="step", Q=64, G=8, r_q=0.5, r_o=0.5, capacity=8192, n_win=32, rollout=3),
        # a micro-batch of the 8B shape under the sequence-level objective with token normalisation and
        # decoupled clip, the longest sequence promised
        dict(q8b, name="qwen3_8b_sequence_ratio", path="loss", mix="long_math", S=13, ratio="sequence",
             aggregation="token_sum", clip_hi=0.28, promise=True, rollout=4),
        # gradient accumulation: one packed row of 8192 tokens at a time, dW added to what is there
        dict(q4b, name="qwen3_4b_packed_row", path="loss", S=6, accumulate=True, rollout=5),
        # short completions of the 8B shape with the logits recomputed in the backward: few tokens
        # against the whole vocabulary
        dict(q8b, name="qwen3_8b_short_recompute", path="loss", mix="short", S=9, recompute=True, rollout=6),
        # float32 (numerics runs of a small model): forward and backward of two or three sequences
        dict(small, name="small_loss_f32", path="loss", dtype="f32", S=3, rollout=7),
        # old-policy log-probs of 8 prompts x 8 completions before the update
        dict(q4b, name="qwen3_4b_logprob", path="logprob", S=64, rollout=8),
        # scoring a single short answer, hidden states of the answer handed over directly
        dict(q8b, name="qwen3_8b_logprob_one", path="logprob", mix="short", S=1, N=333, identity=True, rollout=9),
        # a serving loop scoring a few new tokens without allocating
        dict(q4b, name="qwen3_4b_serve", path="noalloc", mix="short", S=1, N=33, identity=True, rollout=10),
        # a batch of 256 prompts x 16 completions between rollout and update
        dict(name="stress_select_pack", path="select_pack", Q=256, G=16, mix="bimodal", r_q=0.7, r_o=0.7,
             capacity=32768, n_win=32, fixed=False, policy="first_fit", rollout=11),
        # 8.5 K prompts packed once per dataset, rows as long as the longest prompt
        dict(name="prompts_8k5", path="prompts", n=8500, median=90.0, sigma=0.35, lo=16, hi=512, n_win=32,
             policy="first_fit", rollout=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges, never dearer than the largest listed one."""
    path = rng.choice(["step", "step", "loss", "loss", "loss", "logprob", "logprob", "noalloc", "select_pack", "prompts"])
    c = dict(path=path, rollout=rng.randrange(1 << 20))
    if path == "prompts":
        c.update(n=_log_int(rng, 500, 8500), median=round(rng.uniform(80.0, 150.0), 1), sigma=round(rng.uniform(0.3, 0.6), 2),
                 lo=16, hi=rng.choice([512, 1024, 2048]), n_win=rng.choice([8, 16, 32, 64]),
                 policy=rng.choice(["first_fit", "first_fit", "best_fit"]))
        return c
    if path == "select_pack":
        c.update(Q=_log_int(rng, 16, 256), G=rng.choice([4, 8, 16]), mix=rng.choice(["small", "math", "long_math", "bimodal"]),
                 r_q=rng.choice([0.4, 0.5, 0.7]), r_o=rng.choice([0.3, 0.5, 0.7]), capacity=rng.choice([20000, 32768]),
                 n_win=rng.choice([8, 16, 32, 64]), fixed=rng.random() < 0.3,
                 policy=rng.choice(["first_fit", "first_fit", "best_fit"]))
        return c
    if path != "noalloc" and rng.random() < 0.3:
        c.update(dtype="f32", D=_log_int(rng, 64, 1024), V=_log_int(rng, 300, 32000), mix="tiny")
    else:
        c.update(dtype="bf16", D=64 * rng.randint(8, 64), V=_log_int(rng, 30000, 152000),
                 mix=rng.choice(["small", "math", "long_math", "short"]))
    if path == "step":
        c.update(Q=_log_int(rng, 4, 48), G=rng.choice([4, 8]), r_q=rng.choice([0.4, 0.5, 0.6]),
                 r_o=rng.choice([0.3, 0.5]), capacity=rng.choice([8704, 16384]), n_win=rng.choice([16, 32]))
    elif path == "noalloc":
        c.update(mix="short", S=1, N=_log_int(rng, 1, 400), identity=True)
    else:
        c["S"] = _log_int(rng, 1, 48)
        if c["mix"] == "short" and rng.random() < 0.5:
            c.update(S=1, N=_log_int(rng, 5, 900))
        if path == "loss":
            c["accumulate"] = rng.random() < 0.3
            if rng.random() < 0.3:
                c.update(ratio="sequence", promise=True, aggregation=rng.choice(["seq_mean", "token_sum"]), clip_hi=0.28)
            elif c["dtype"] == "bf16" and rng.random() < 0.2:
                c["recompute"] = True
        else:
            c["identity"] = rng.random() < 0.3
    while work(c)["flops"] > (3e11 if c["dtype"] == "f32" else 5e14):     # (float32 runs at a twentieth of the bf16 rate)
        key = "Q" if path == "step" else "S"
        c[key] = max(1, c[key] // 2)
    return c


# ---- sizes: everything here follows from the case alone ---------------------------------------
def _lengths(rng, law, shape):
    if law[0] == "uniform":
        return rng.integers(law[1], law[2] + 1, size=shape)
    if law[0] == "lognormal":
        return np.clip(np.rint(rng.lognormal(math.log(law[1]), law[2], size=shape)), law[3], law[4]).astype(np.int64)
    pick = rng.random(size=shape) < 0.5
    return np.where(pick, rng.integers(law[1], law[2] + 1, size=shape), rng.integers(law[3], law[4] + 1, size=shape))


def _rollouts(c):
    """Q prompts x G completions after rollout: lengths, 0/1 rewards, last epoch's scores, pruning uniforms."""
    rng = np.random.default_rng([c["rollout"], 0xD990])
    Q, G = c["Q"], c["G"]
    pr, law = MIXES[c["mix"]]
    r = dict(prompt_len=rng.integers(pr[0], pr[1] + 1, size=Q), comp_len=_lengths(rng, law, (Q, G)))
    r["rewards"] = (rng.random((Q, G)) < rng.beta(0.5, 0.5, size=Q)[:, None]).astype(np.float32)
    r["hist"], r["u_prompt"] = rng.random(Q, dtype=np.float32), rng.random(Q, dtype=np.float32)
    r["u_comp"] = rng.random((Q, G), dtype=np.float32)
    return r


def _sequences(c):
    """Prompt and completion lengths of S packed sequences."""
    rng = np.random.default_rng([c["rollout"], 0x5E9])
    pr, law = MIXES[c["mix"]]
    pl, cl = rng.integers(pr[0], pr[1] + 1, size=c["S"]), _lengths(rng, law, c["S"])
    if c.get("N"):
        cl = np.full(1, c["N"])
    if c.get("identity"):
        pl = np.zeros_like(pl)
    return pl, cl


def _kept_tokens(c):
    """(packed tokens, loss tokens) of the sequences that survive pruning in a `step` case."""
    r, G = _rollouts(c), c["G"]
    dev = np.abs(G * r["rewards"].astype(np.float64) - r["rewards"].sum(axis=1, keepdims=True))
    cand = G * dev <= dev.sum(axis=1, keepdims=True)
    keep = ~(cand & (r["u_comp"] < np.float32(c["r_o"])))
    low = np.argsort(r["hist"], kind="stable")[: c["Q"] // 2]
    keep[low[r["u_prompt"][low] < np.float32(c["r_q"])]] = False
    cl = r["comp_len"][keep]
    return int((r["prompt_len"][:, None] + r["comp_len"])[keep].sum()), int(cl.sum())


def work(c):
    if c["path"] == "prompts":
        return {"bytes": 4 * c["n"] * 5, "flops": 0}
    if c["path"] == "select_pack":
        Q, G = c["Q"], c["G"]
        r = _rollouts(c)
        # inputs; adv, masks, weights; order and offsets; the loss positions (about half survive pruning)
        return {"bytes": Q * G * (16 + 25 + 24) + Q * 40 + 4 * int(r["comp_len"].sum()) // 2, "flops": 0}
    es = 4 if c["dtype"] == "f32" else 2
    D, V = c["D"], c["V"]
    if c["path"] == "step":
        T, N = _kept_tokens(c)
    else:
        pl, cl = _sequences(c)
        T, N = int(pl.sum() + cl.sum()), int(cl.sum())
    read = N * D * es + V * D * es
    if c["path"] in ("logprob", "noalloc"):
        return {"bytes": read + 16 * N, "flops": 2.0 * D * V * N}
    dw = V * D * 4 * (2 if c.get("accumulate") else 1)
    return {"bytes": read + T * D * es + dw + 20 * N, "flops": 6.0 * D * V * N}


def tolerance(c):
    """About four times what the library's outputs are off from the same formulas in float64 (the listed cases, the
    large ones on a few of their sequences): log-probs and lse 7e-8 (2.3e-7 at worst); bf16 gradients 2.4e-3
    (exponentials and row-scaled operands rounded to bf16; single entries of the rows of frequent tokens, where
    large terms cancel, are off by up to 0.8 of the array's root mean square); float32 gradients 3.3e-6 (2.7e-5 at
    worst). Whole numbers (masks, counts, order, offsets) are the same or wrong."""
    if c["path"] == "prompts":
        return "exact"
    if c["path"] == "select_pack":
        return {"rel": 1e-6}                       # float64 inside, one rounding to float32
    if c["path"] in ("logprob", "noalloc"):
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 1e-2, "max": 0.95} if c["dtype"] == "bf16" else {"rel": 1.3e-5, "max": 2e-4}


# ---- what a program holds before the call ------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 65537 + salt)
    return g


def _dev(a, dtype):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV).to(dtype).contiguous()


def _normal(g, rows, cols, std, dtype):
    out = torch.empty((rows, cols), dtype=dtype, device=DEV)
    for r in range(0, rows, 1 << 16):              # in pieces: the float32 draw of the largest does not double the state
        n = min(rows - r, 1 << 16)
        out[r:r + n] = (torch.randn((n, cols), generator=g, device=DEV) * std).to(dtype)
    return out


def _model(c, seed, T):
    """Hidden states, vocabulary matrix and token ids (Zipf over the large vocabularies, else uniform)."""
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    g, V = _gen(seed, 1), c["V"]
    H = _normal(g, T, c["D"], 1.0, dt)
    W = _normal(g, V, c["D"], 0.05 if V <= 1000 else 0.02, dt)
    if V > 100000:
        p = torch.arange(1, V + 1, device=DEV, dtype=torch.float64) ** -1.1
        cdf = torch.cumsum(p / p.sum(), 0)
        ranks = torch.searchsorted(cdf, torch.rand(T, generator=g, device=DEV, dtype=torch.float64)).clamp(max=V - 1)
        ids = torch.randperm(V, generator=g, device=DEV)[ranks].to(torch.int32)
    else:
        ids = torch.randint(0, V, (T,), generator=g, device=DEV, dtype=torch.int32)
    return H, W, ids


def _head_buffers(c, s, N, S, want):
    """Workspace, gradients and outputs that a training loop keeps from step to step, and the behaviour and
    reference log-probs of these inputs."""
    H, W = s["H"], s["W"]
    s["ws"] = P.alloc_workspace(P.dppo_workspace_bytes(H.shape[0], N, c["D"], c["V"], 0 if c["dtype"] == "f32" else 1, want), DEV)
    if want == 0:
        return
    base, _ = P.dppo_token_logprob(H, W, s["ids"], s["loss_pos"], want_lse=False, ws=s["ws"])
    g = _gen(s["seed"], 2)
    s["logp_old"] = base + NOISE * torch.randn(N, generator=g, device=DEV)
    s["logp_ref"] = base + NOISE * torch.randn(N, generator=g, device=DEV)
    s["dH"] = torch.empty_like(H)
    s["dW"] = (_normal(g, c["V"], c["D"], 1e-6, torch.float32) if c.get("accumulate")
               else torch.empty((c["V"], c["D"]), device=DEV))
    f = dict(dtype=torch.float32, device=DEV)
    s["out"] = dict(loss=torch.empty(1, **f), logp=torch.empty(N, **f), seq_loss=torch.empty(S, **f), stats=torch.empty(4, **f))
    s["status"] = torch.zeros(1, dtype=torch.int32, device=DEV)


def _batch(r, order=None):
    """A batch of rollouts on the GPU, its prompts in arrival order `order`."""
    o = np.arange(len(r["prompt_len"])) if order is None else order
    G = r["comp_len"].shape[1]
    return dict(rewards=_dev(r["rewards"][o], torch.float32), hist=_dev(r["hist"][o], torch.float32),
                u_prompt=_dev(r["u_prompt"][o], torch.float32), u_comp=_dev(r["u_comp"][o], torch.float32),
                prompt_len=_dev(np.repeat(r["prompt_len"][o], G), torch.int32),
                comp_len=_dev(r["comp_len"][o].reshape(-1), torch.int32), lp_cap=int(r["comp_len"].sum()))


def _select(c, b):
    return P.dppo_select(b["rewards"], b["hist"], b["u_prompt"], b["u_comp"], c["r_q"], c["r_o"],
                         fixed_count=c.get("fixed", False), device=DEV)


def _pack(c, b, keep):
    return P.dppo_pack(b["prompt_len"], b["comp_len"], keep.reshape(-1), c["capacity"], c["n_win"],
                       loss_pos_capacity=b["lp_cap"], device=DEV, policy=c.get("policy", "first_fit"))


def _pack_prompts(c, lens):
    return P.dppo_pack(lens, None, None, 0, c["n_win"], loss_pos_capacity=0, device=DEV, policy=c["policy"])


def _arrival_order(n, seed, rows_of):
    """An arrival order made from the seed whose packing has as many rows as the order 0 .. n-1, so that the
    arrays of all seeds are of one size."""
    want = rows_of(np.arange(n))
    rng = np.random.default_rng([seed, 0xA881])
    for _ in range(400):
        order = rng.permutation(n)
        if rows_of(order) == want:
            return order
    raise RuntimeError("no arrival order of %d with %r rows" % (n, want))


def prepare(case, seed):
    c, s = case, dict(case=case, seed=int(seed))
    if c["path"] == "prompts":
        rng = np.random.default_rng([c["rollout"], 0xDA7A])
        lens = _lengths(rng, ("lognormal", c["median"], c["sigma"], c["lo"], c["hi"]), c["n"])
        order = _arrival_order(c["n"], s["seed"], lambda o: _pack_prompts(c, _dev(lens[o], torch.int32))["n_rows"])
        s["prompt_len"] = _dev(lens[order], torch.int32)
        return s
    if c["path"] == "select_pack":
        r = _rollouts(c)

        def rows(o):
            b = _batch(r, o)
            pk = _pack(c, b, _select(c, b)["keep_comp"])
            return pk["S"], pk["N"], pk["n_rows"]

        order = _arrival_order(c["Q"], s["seed"], rows)
        s.update(_batch(r, order))
        s["index"] = torch.as_tensor(order, device=DEV).to(torch.int32)
        s["scores"] = torch.zeros(c["Q"], device=DEV)
        return s
    if c["path"] == "step":
        s.update(_batch(_rollouts(c)))
        pk = _pack(c, s, _select(c, s)["keep_comp"])
        T, N, s["loss_pos"] = pk["T"], pk["N"], pk["loss_pos"]
        s["H"], s["W"], s["ids"] = _model(c, s["seed"], T)
        _head_buffers(c, s, N, c["Q"] * c["G"], 1)
        return s
    pl, cl = _sequences(c)
    cu = np.concatenate([[0], np.cumsum(pl + cl)])
    T, N = int(cu[-1]), int(cl.sum())
    s["H"], s["W"], s["ids"] = _model(c, s["seed"], T)
    s["loss_pos"] = None if c.get("identity") else _dev(
        np.concatenate([np.arange(a + p - 1, a + p + n - 1) for a, p, n in zip(cu, pl, cl)]), torch.int32)
    if c["path"] == "noalloc":
        s["logp"], s["lse"] = torch.empty(N, device=DEV), torch.empty(N, device=DEV)
        return s
    if c["path"] == "loss":
        s["loss_cu"] = _dev(np.concatenate([[0], np.cumsum(cl)]), torch.int32)
        g = _gen(seed, 3)
        s["seq_adv"] = torch.randn(len(cl), generator=g, device=DEV)
        s["seq_coef"] = torch.full((len(cl),), 1.0 / len(cl), device=DEV)
        if c.get("aggregation") == "token_sum":
            s["seq_coef"] /= float(cl.mean())
        s["max_seq"] = int(cl.max()) if c.get("promise") else 0
    _head_buffers(c, s, N, c["S"], 0 if c["path"] == "logprob" else 2 if c.get("promise") else 1)
    return s


# ---- one pass ----------------------------------------------------------------------------------
def _loss(c, s, loss_pos, loss_cu, adv, coef):
    return P.dppo_loss_fwd_bwd(s["H"], s["W"], s["ids"], loss_pos, loss_cu, adv, coef, s["logp_old"], s["logp_ref"],
                               CLIP, c.get("clip_hi", CLIP), BETA, dW=s["dW"], dH=s["dH"], ws=s["ws"], out=s["out"],
                               accumulate_dW=c.get("accumulate", False), recompute_logits=c.get("recompute", False),
                               ratio_level=c.get("ratio", "token"), aggregation=c.get("aggregation", "seq_mean"),
                               status=s["status"], max_seq_tokens=s.get("max_seq", 0))


def run(s):
    c = s["case"]
    if c["path"] == "step":
        sel = _select(c, s)
        pk = _pack(c, s, sel["keep_comp"])
        adv = P.dppo_gather_f32(pk["order"], sel["adv"])
        coef = P.dppo_gather_f32(pk["order"], sel["coef"])
        return _loss(c, s, pk["loss_pos"], pk["loss_cu"], adv, coef)
    if c["path"] == "loss":
        return _loss(c, s, s["loss_pos"], s["loss_cu"], s["seq_adv"], s["seq_coef"])
    if c["path"] == "logprob":
        return P.dppo_token_logprob(s["H"], s["W"], s["ids"], s["loss_pos"], ws=s["ws"])
    if c["path"] == "noalloc":
        P.dppo_token_logprob_noalloc(s["H"], s["W"], s["ids"], None, s["logp"], s["lse"])
        return s["logp"], s["lse"]
    if c["path"] == "prompts":
        return _pack_prompts(c, s["prompt_len"])
    sel = _select(c, s)
    scores = P.dppo_history_update(s["scores"], s["index"], sel["keep_prompt"], sel["mean_abs_adv"])
    weights = P.dppo_token_norm_coef(sel["coef"], s["comp_len"])
    pk = _pack(c, s, sel["keep_comp"])
    return dict(select=sel, scores=scores, pack=pk, adv=P.dppo_gather_f32(pk["order"], sel["adv"]),
                coef=P.dppo_gather_f32(pk["order"], weights))
