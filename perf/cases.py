"""The workloads this library is timed on: the calls of one training step of probabilistic chunk masking, over the
sizes and options its users run them with.

A case is a dict of plain values.  `listed()` names the fixed ones, `draw(rng)` makes one more of the same ranges;
`prepare(case, seed)` makes on the GPU what a training program holds before the call, `run(state)` is one pass through
the public entry points, `work(case)` the bytes and operations the pass cannot do without, `tolerance(case)` how far
another correct implementation may be from it, and `exact(case, seed)` the pass in 64 bits with plain torch.

Three kinds of pass:
  select  pcm_score_phases, pcm_update_keep_probs, pcm_sample_chunks; with "label" pcm_label_phases in front and
          pcm_importance_weights, pcm_kept_phase_counts behind
  step    grpo_masked_actor_step (forward and backward, or with "grads" false the log-probabilities alone)
  update  pcm_adamw_clip_step and, with "pack", pcm_pack_head_weights
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2605_16154_amd as pcm

EPS_LOW, EPS_HIGH = 0.2, 0.4          # clip thresholds of the training runs
ADV_EPS = 1e-6
P_MIN = 0.1
WEIGHTS = ("Wg", "Wu", "Wd", "Wo")


# ---- the cases ---------------------------------------------------------------------------------

def _select(name, groups, N, K, B, L=8, D=7, G=8, selector="pcm", label=False, ragged=False, collapsed=0.0):
    return dict(name=name, kind="select", groups=groups, G=G, N=N, K=K, B=B, L=L, D=D, selector=selector, label=label,
                ragged=ragged, collapsed=collapsed)


def _step(name, dtype, groups, N, B, d, ff, V=256, A=56, G=8, drift=0.1, entropy=0.0, token_mean=False, chunk_ratio=False,
          composed=False, packed=False, sumsq=False, grads=True, ragged=False):
    return dict(name=name, kind="step", dtype=dtype, groups=groups, G=G, N=N, B=B, A=A, d=d, ff=ff, V=V, drift=drift,
                entropy=entropy, token_mean=token_mean, chunk_ratio=chunk_ratio, composed=composed, packed=packed,
                sumsq=sumsq, grads=grads, ragged=ragged)


def _update(name, d, ff, V=256, bf16=True, norm_given=False, pack=True):
    return dict(name=name, kind="update", d=d, ff=ff, V=V, bf16=bf16, norm_given=norm_given, pack=pack)


def listed():
    return [
        # the selection of the tiny instance: 16 trajectories, all launch latency
        _select("select-tiny", 2, N=32, K=4, B=6),
        # the long-horizon selection: 512 trajectories of up to 256 chunks, a quarter of the groups collapsed
        _select("select-long", 64, N=256, K=12, B=24, ragged=True, collapsed=0.25),
        # the selection from raw gripper commands with fixed per-phase budgets, estimator weights and the logged
        # allocation, at the larger batch of the multi-task instance
        _select("select-labelled", 32, N=128, K=5, B=16, selector="stratified", label=True, ragged=True),
        # the step of the tiny fp32 instance (the accuracy reference users validate a run against)
        _step("step-f32-tiny", "f32", 2, N=32, B=6, d=256, ff=1024),
        # the same at a mid-sized head with the entropy bonus of the training runs
        _step("step-f32-mid", "f32", 4, N=32, B=6, d=1024, ff=2816, entropy=1e-3, token_mean=True, ragged=True),
        # a small bf16 head, a few chunks per trajectory, the kept list shorter than its buffer
        _step("step-bf16-small", "bf16", 1, N=16, B=5, d=512, ff=768, ragged=True),
        # log-probabilities of one trajectory's kept chunks under the 7B policy's head (the old-policy pass)
        _step("logp-bf16-one", "bf16", 1, G=1, N=64, B=12, d=4096, ff=11008, packed=True, grads=False),
        # one task group at the 7B head, with entropy bonus and token mean
        _step("step-bf16-group", "bf16", 1, N=64, B=12, d=4096, ff=11008, packed=True, entropy=1e-3, token_mean=True,
              ragged=True),
        # two groups with one ratio per chunk
        _step("step-bf16-chunk-ratio", "bf16", 2, N=64, B=12, d=4096, ff=11008, packed=True, drift=0.3, chunk_ratio=True),
        # the masked step the headline figure is quoted on, the policy some way from the one that made the rollouts
        _step("step-bf16-masked", "bf16", 8, N=64, B=12, d=4096, ff=11008, packed=True, drift=1.0, sumsq=True),
        # the unmasked step it is compared with: every chunk kept, near on-policy
        _step("step-bf16-unmasked", "bf16", 8, N=64, B=64, d=4096, ff=11008, packed=True),
        # clipping, AdamW and the re-laid-out weights of the 7B head
        _update("update-7b-head", 4096, 11008),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["select", "step-f32", "step-bf16", "step-bf16", "logp-bf16", "update"])
    if kind == "select":
        label = rng.random() < 0.4
        N = _log_int(rng, 16, 256)
        case = _select("", _log_int(rng, 1, 64), N=N, K=5 if label else rng.randint(2, min(12, N)),
                       B=min(N, rng.randint(2, 24)), G=rng.choice([4, 5, 8, 10]), L=rng.choice([4, 5, 8]),
                       D=rng.choice([3, 7]), selector=rng.choice(["pcm", "pcm", "random", "top_phase", "stratified"]),
                       label=label, ragged=rng.random() < 0.6, collapsed=rng.choice([0.0, 0.25]))
    elif kind == "step-f32":
        case = _step("", "f32", rng.randint(1, 4), N=rng.randint(8, 32), B=rng.randint(2, 6), d=_log_int(rng, 64, 1024),
                     ff=_log_int(rng, 128, 2816), V=rng.choice([101, 256, 256, 512]), A=rng.choice([15, 56, 56]),
                     drift=rng.choice([0.1, 1.0]), entropy=rng.choice([0.0, 1e-3]), token_mean=rng.random() < 0.5,
                     composed=rng.random() < 0.25, ragged=rng.random() < 0.5)
    elif kind == "update":
        bf16 = rng.random() < 0.7
        d, ff = (256 * _log_int(rng, 1, 16), 256 * _log_int(rng, 1, 43)) if bf16 else (_log_int(rng, 64, 1024), _log_int(rng, 128, 2816))
        case = _update("", d, ff, bf16=bf16, norm_given=rng.random() < 0.5, pack=bf16)
    else:
        grads = kind == "step-bf16"
        d, ff = 256 * _log_int(rng, 1, 16), 256 * _log_int(rng, 1, 43)
        composed = rng.random() < 0.2
        listed_rows = rng.random() < 0.5
        case = _step("", "bf16", _log_int(rng, 1, 8), G=rng.choice([1, 4, 8]), N=rng.randint(12, 64), B=rng.randint(1, 12), d=d,
                     ff=ff, A=rng.choice([4, 16, 56, 56, 56]), drift=rng.choice([0.1, 1.0]),
                     entropy=0.0 if listed_rows else 1e-3, token_mean=rng.random() < 0.5, composed=composed,
                     packed=not composed and rng.random() < 0.7, sumsq=grads and not composed and rng.random() < 0.5,
                     grads=grads, ragged=rng.random() < 0.5)
    del case["name"]
    return case


# ---- inputs ------------------------------------------------------------------------------------

def _generators(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return np.random.default_rng(seed), g


def _to_gpu(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _rewards(rng, groups, G, collapsed=0.0):
    r = (rng.random((groups, G)) < 0.5).astype(np.uint8)
    for g in range(groups):
        if rng.random() < collapsed:
            r[g] = rng.integers(0, 2)
        elif G > 1 and r[g].min() == r[g].max():
            r[g, rng.integers(0, G)] ^= 1
    return r.reshape(-1)


def _phases(rng, T, N, K):
    """K contiguous phases per trajectory, boundaries drawn uniformly."""
    cuts = np.sort(rng.integers(1, N + 1, size=(T, K - 1)), axis=1)
    return (np.arange(N)[None, :, None] >= cuts[:, None, :]).sum(axis=2).astype(np.uint8)


def _select_inputs(case, seed):
    rng, gen = _generators(seed)
    groups, G, N, K, L, D = (case[k] for k in ("groups", "G", "N", "K", "L", "D"))
    T, A = groups * G, L * D
    reward, phase = _rewards(rng, groups, G, case["collapsed"]), _phases(rng, T, N, K)
    n_chunks = rng.integers(N // 3, N + 1, size=T).astype(np.int32) if case["ragged"] else np.full(T, N, np.int32)
    # per (group, phase) mean action; successes and failures differ by half a unit in one phase out of three
    centre = rng.uniform(-0.5, 0.5, size=(groups, K, A))
    gap = 0.5 * (rng.random((groups, K)) < 0.34)
    g = np.repeat(np.arange(groups), G)
    shift = (reward.astype(np.float64) - 0.5)[:, None] * gap[g[:, None], phase]
    mean = _to_gpu(centre.astype(np.float32))[_to_gpu(g)[:, None], _to_gpu(phase.astype(np.int64))] + _to_gpu(shift.astype(np.float32))[..., None]
    actions = (mean + 0.1 * torch.randn((T, N, A), generator=gen, device="cuda")).clamp_(-1.0, 1.0)
    if case["label"]:   # gripper command (last dimension): open, one held grasp with a few drop-outs, open
        start, hold = rng.integers(1, max(2, N // 2), size=T), rng.integers(1, max(2, N // 2), size=T)
        k = np.arange(N)[None, :]
        held = (k >= start[:, None]) & (k < (start + hold)[:, None])
        p_close = np.where(held, 0.95, 0.08)
        closed = rng.random((T, N, L)) < p_close[:, :, None]
        actions.view(T, N, L, D)[..., D - 1] = _to_gpu(np.where(closed, 1.0, -1.0).astype(np.float32))
    return dict(actions=actions.contiguous(), phase=_to_gpu(phase), reward=_to_gpu(reward), n_chunks=_to_gpu(n_chunks))


def _head_logp(x, w, tokens, out_blocks):
    """log-probabilities of `tokens` under the head, row block by row block (x already in the working precision)."""
    for r0 in range(0, x.shape[0], out_blocks):
        r1 = min(x.shape[0], r0 + out_blocks)
        a = torch.nn.functional.silu(x[r0:r1] @ w["Wg"]) * (x[r0:r1] @ w["Wu"])
        z = (a @ w["Wd"]) @ w["Wo"]
        yield r0, r1, torch.log_softmax(z, dim=1).gather(1, tokens[r0:r1, None])[:, 0]


def _away_from_thresholds(delta, margin):
    """log-ratios moved out of a margin around the two clip thresholds (a ratio on a threshold is a coin toss)."""
    for thr in (math.log1p(-EPS_LOW), math.log1p(EPS_HIGH)):
        near = (delta - thr).abs() < margin
        delta = torch.where(near, thr + torch.where(delta >= thr, 2 * margin, -2 * margin).to(delta.dtype), delta)
    return delta


def _step_inputs(case, seed):
    rng, gen = _generators(seed)
    groups, G, N, B, A, d, ff, V = (case[k] for k in ("groups", "G", "N", "B", "A", "d", "ff", "V"))
    T, B = groups * G, min(B, N)
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    reward = _rewards(rng, groups, G).reshape(groups, G).astype(np.float64)
    sd = reward.std(axis=1, keepdims=True)
    adv = np.where(sd > 0, (reward - reward.mean(axis=1, keepdims=True)) / (sd + ADV_EPS), 1.0).astype(np.float32).reshape(-1)
    kept = []
    for i in range(T):
        n = int(rng.integers((B + 1) // 2, B + 1)) if case["ragged"] else B
        kept += [i * N + int(k) for k in np.sort(rng.permutation(N)[:n])]
    capacity = T * B
    kept_idx = np.zeros(capacity, np.int32)
    kept_idx[:len(kept)] = kept
    rows_all = T * N * A
    hidden = torch.empty((rows_all, d), dtype=dtype, device="cuda")
    for r0 in range(0, rows_all, 1 << 15):
        r1 = min(rows_all, r0 + (1 << 15))
        hidden[r0:r1] = torch.randn((r1 - r0, d), generator=gen, device="cuda").to(dtype)
    # weights N(0, 0.02) at the widths of the 7B head; scaled at narrower ones so that logits stay of order one
    std = {"Wg": 1.28 / math.sqrt(d), "Wu": 1.28 / math.sqrt(d), "Wd": 2.1 / math.sqrt(ff), "Wo": 1.28 / math.sqrt(d)}
    shape = {"Wg": (d, ff), "Wu": (d, ff), "Wd": (ff, d), "Wo": (d, V)}
    w = {k: (torch.randn(shape[k], generator=gen, device="cuda") * std[k]).to(dtype) for k in WEIGHTS}
    tokens = torch.randint(0, min(V, 256), (rows_all,), generator=gen, device="cuda", dtype=torch.int32).to(torch.uint8)
    # logp_old of the kept rows: what the current head gives minus a log-ratio of the stated spread
    logp_old = torch.full((rows_all,), -5.5, device="cuda")
    if case["grads"]:
        rows = (_to_gpu(np.asarray(kept, np.int64))[:, None] * A + torch.arange(A, device="cuda")[None, :]).reshape(-1)
        margin = 1e-3 if dtype == torch.float32 else 0.08
        if case["chunk_ratio"]:
            per_chunk = _away_from_thresholds(case["drift"] * torch.randn((len(kept),), generator=gen, device="cuda"), 0.02)
            noise = 0.05 * torch.randn((len(kept), A), generator=gen, device="cuda")
            delta = (per_chunk[:, None] / A + noise - noise.mean(dim=1, keepdim=True)).reshape(-1)
        else:
            delta = _away_from_thresholds(case["drift"] * torch.randn((rows.shape[0],), generator=gen, device="cuda"), margin)
        wf = {k: w[k].float() for k in WEIGHTS}
        tok = tokens[rows].long()
        for r0, r1, lp in _head_logp(hidden[rows].float() if rows.shape[0] <= 1 << 15 else _Rows(hidden, rows), wf, tok, 1 << 13):
            logp_old[rows[r0:r1]] = lp - delta[r0:r1]
    return dict(hidden=hidden, tokens=tokens, logp_old=logp_old, adv=_to_gpu(adv), kept_idx=_to_gpu(kept_idx),
                n_kept=_to_gpu(np.array([len(kept)], np.int32)), n_kept_host=len(kept), kept_host=np.asarray(kept, np.int64),
                capacity=capacity, T=T, **w)


class _Rows:
    """Rows of a matrix by number, converted a block at a time."""

    def __init__(self, x, rows, dtype=torch.float32):
        self.x, self.rows, self.dtype, self.shape = x, rows, dtype, (rows.shape[0], x.shape[1])

    def __getitem__(self, block):
        return self.x[self.rows[block]].to(self.dtype)


def _update_inputs(case, seed):
    _, gen = _generators(seed)
    d, ff, V = case["d"], case["ff"], case["V"]
    shapes = [(d, ff), (d, ff), (ff, d), (d, V)]
    rand = lambda s, scale: torch.randn(s, generator=gen, device="cuda") * scale
    w = [rand(s, 0.02) for s in shapes]
    grads = [rand(s, 1e-3) for s in shapes]
    m = [rand(s, 5e-4) for s in shapes]
    v = [rand(s, 1e-3).square_() for s in shapes]
    return w, grads, m, v


# ---- what a program holds, and one pass --------------------------------------------------------

def prepare(case, seed):
    if case["kind"] == "select":
        st = dict(case=case, **_select_inputs(case, seed))
        T, N, K, B, A = case["groups"] * case["G"], case["N"], case["K"], case["B"], case["L"] * case["D"]
        z = lambda n, dt: torch.zeros(n, dtype=dt, device="cuda")
        n_max = T * min(B, N)
        st.update(keep=pcm.pcm_state_init(K), p=z(K, torch.float64), labels=z((T, N), torch.uint8),
                  score=(z(K, torch.float64), z(K, torch.uint8), z(T, torch.float32), z(T, torch.uint8)),
                  sample=(z(n_max, torch.int32), z(T + 1, torch.int32), z(1, torch.int32)),
                  weights=z(n_max, torch.float32), counts=(z(K, torch.int32), z(K, torch.int32)))
        return st
    if case["kind"] == "update":
        w, grads, m, v = _update_inputs(case, seed)
        st = dict(case=case, w=w, grads=grads, m=m, v=v, norm=torch.zeros(1, device="cuda"), sumsq=None, lowp=None, packed=None)
        if case["norm_given"]:
            st["sumsq"] = sum(g.double().square().sum() for g in grads).reshape(1)
        if case["bf16"]:
            st["lowp"] = [x.to(torch.bfloat16) for x in w]
        if case["pack"]:
            st["packed"] = pcm.pcm_pack_head_weights(*st["lowp"])
        return st
    st = dict(case=case, **_step_inputs(case, seed))
    rows, d, ff, V, hdt = st["capacity"] * case["A"], case["d"], case["ff"], case["V"], st["hidden"].dtype
    z = lambda shape, dt: torch.zeros(shape, dtype=dt, device="cuda")
    out = dict(loss=z(1, torch.float32), logp=z(rows, torch.float32), stats=z(5, torch.float32))
    if case["grads"]:
        out.update(dWg=z((d, ff), torch.float32), dWu=z((d, ff), torch.float32), dWd=z((ff, d), torch.float32),
                   dWo=z((d, V), torch.float32), dX=z((rows, d), hdt))
    if case["sumsq"]:
        out["grad_sumsq"] = z(1, torch.float64)
    st["out"] = out
    st["packed_weights"] = pcm.pcm_pack_head_weights(*(st[k] for k in WEIGHTS)) if case["packed"] else None
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "select":
        phase, n_chunks, K, G = st["phase"], st["n_chunks"], case["K"], case["G"]
        if case["label"]:
            phase = pcm.pcm_label_phases(st["actions"], n_chunks, case["L"], case["D"], out=st["labels"])
        C, valid, adv, active = pcm.pcm_score_phases(st["actions"], phase, st["reward"], n_chunks, case["groups"], G, K,
                                                     ADV_EPS, out=st["score"])
        p = pcm.pcm_update_keep_probs(st["keep"], C, valid, P_MIN, 1, keep_probs_out=st["p"])   # refreshed on every pass
        kept, offsets, n_kept = pcm.pcm_sample_chunks(p, phase, n_chunks, active, case["B"], 17, 3, out=st["sample"],
                                                      selector=case["selector"])
        out = [C, valid, adv, active, p, kept, offsets, n_kept]
        if case["label"]:
            out.append(phase)
            out.append(pcm.pcm_importance_weights(phase, n_chunks, kept, offsets, K, out=st["weights"]))
            out += list(pcm.pcm_kept_phase_counts(phase, n_chunks, active, kept, n_kept, K, out=st["counts"]))
        return out
    if case["kind"] == "update":
        norm = pcm.pcm_adamw_clip_step(st["grads"], st["w"], st["m"], st["v"], 100, weights_bf16=st["lowp"],
                                       grad_norm_out=st["norm"], grad_sumsq=st["sumsq"])
        out = [norm, *st["w"], *st["m"], *st["v"]]
        if case["bf16"]:
            out += st["lowp"]
        if case["pack"]:
            out.append(pcm.pcm_pack_head_weights(*st["lowp"], out=st["packed"]).view(torch.bfloat16))
        return out
    out = pcm.grpo_masked_actor_step(
        st["hidden"], st["tokens"], st["logp_old"], st["adv"], st["kept_idx"], st["n_kept"], st["T"], case["N"], case["A"],
        st["Wg"], st["Wu"], st["Wd"], st["Wo"], EPS_LOW, EPS_HIGH, 1.0 if case["token_mean"] else 1.0 / st["T"],
        want_grads=case["grads"], want_dX=case["grads"], out=st["out"], token_mean=case["token_mean"],
        entropy_coef=case["entropy"], chunk_ratio=case["chunk_ratio"], composed_head=case["composed"],
        packed_weights=st["packed_weights"], grad_sumsq=case["sumsq"])
    if case["grads"]:
        return dict(out)
    return dict(logp=out["logp"])      # the old-policy pass: loss and statistics are of no use to it


# ---- what the pass cannot do without -----------------------------------------------------------

def _normal_cdf(x):
    return 0.5 * (1.0 + math.erf(x / math.sqrt(2.0)))


def _share_with_gradient(case):
    """Expected share of rows the clip lets through (half of them with a positive advantage)."""
    if case["entropy"] != 0.0 or case["G"] == 1:
        return 1.0
    lo, hi = math.log1p(-EPS_LOW) / case["drift"], math.log1p(EPS_HIGH) / case["drift"]
    return 0.5 * _normal_cdf(hi) + 0.5 * (1.0 - _normal_cdf(lo))


def work(case):
    if case["kind"] == "select":
        T, N, A = case["groups"] * case["G"], case["N"], case["L"] * case["D"]
        valid = T * N * (2.0 / 3.0 if case["ragged"] else 1.0)
        kept = T * min(case["B"], N)
        return {"bytes": int(valid * (4 * A + 1) + T * (1 + 4 + 4 + 1 + 4) + kept * (8 if case["label"] else 4)
                             + (T * N if case["label"] else 0)),
                "flops": int(valid * A * 2)}
    if case["kind"] == "update":
        n = 2 * case["d"] * case["ff"] + case["ff"] * case["d"] + case["d"] * case["V"]
        per = 28 + (2 if case["bf16"] else 0) + (2 if case["pack"] else 0)      # g, w, m, v read; w, m, v written
        return {"bytes": n * per, "flops": n * 14}
    d, ff, V, e = case["d"], case["ff"], case["V"], 4 if case["dtype"] == "f32" else 2
    kept = case["groups"] * case["G"] * min(case["B"], case["N"]) * (0.76 if case["ragged"] else 1.0)
    rows = kept * case["A"]
    n_w = 3 * d * ff + d * V
    byt = rows * (d * e + 9) + n_w * e + rows * 4
    if case["composed"]:
        forward, once = 4 * d * ff + 2 * ff * V, 2 * ff * d * V
        backward = 2 * ff * V + 2 * ff * V + 4 * d * ff + 4 * d * ff
    else:
        forward, once, backward = 6 * d * ff + 2 * d * V, 0, 2 * (6 * d * ff + 2 * d * V)
    flops = rows * forward + once
    if case["grads"]:
        flops += rows * _share_with_gradient(case) * backward + 2 * once
        byt += n_w * 4 + rows * d * e
    return {"bytes": int(byt), "flops": int(flops)}


def tolerance(case):
    if case["kind"] == "select":
        return "exact"
    # measured against exact(), times about four.  fp32 steps: gradients 3e-6 to 5e-6, the loss (a sum of terms of both
    # signs) 2e-5; bf16 steps: gradients 8.5e-3; updates: the bf16 copy of the weights 1.7e-3, fp32 state 4e-8
    if case["kind"] == "update":
        return {"rel": 4e-3} if case["bf16"] else {"rel": 1e-6}
    return {"rel": 8e-5} if case["dtype"] == "f32" else {"rel": 3.5e-2}


# ---- the pass in 64 bits -----------------------------------------------------------------------

def exact(case, seed):
    if case["kind"] == "select":
        return _exact_select(case, seed)
    if case["kind"] == "update":
        return _exact_update(case, seed)
    return _exact_step(case, seed)


def _exact_select(case, seed):
    inp = _select_inputs(case, seed)
    groups, G, N, K = case["groups"], case["G"], case["N"], case["K"]
    r = inp["reward"].cpu().numpy().reshape(groups, G) != 0
    mu = r.mean(axis=1, keepdims=True)
    mixed = (mu > 0) & (mu < 1)
    adv = np.where(mixed, (r - mu) / (np.sqrt(mu * (1 - mu)) + ADV_EPS), 0.0).reshape(-1)
    active = np.repeat(mixed[:, 0], G).astype(np.uint8)
    C = valid = p = None
    if not case["label"]:       # with labels the phases are an output of the pass
        x = inp["actions"].double()
        ph = inp["phase"].long()
        ok = torch.arange(N, device="cuda")[None, :] < inp["n_chunks"][:, None]
        out = torch.from_numpy(r.reshape(-1)).cuda().long()
        g = torch.arange(groups, device="cuda").repeat_interleave(G)
        slot = ((g * 2 + out)[:, None] * K + ph)[ok]
        n = torch.zeros(groups * 2 * K, dtype=torch.float64, device="cuda").index_add_(0, slot, torch.ones_like(slot, dtype=torch.float64))
        s = torch.zeros((groups * 2 * K, x.shape[2]), dtype=torch.float64, device="cuda").index_add_(0, slot, x[ok])
        n, mean = n.view(groups, 2, K), (s / n.clamp(min=1.0)[:, None]).view(groups, 2, K, -1)
        pair_ok = (n[:, 0] > 0) & (n[:, 1] > 0) & torch.from_numpy(mixed).cuda()
        pair = (mean[:, 1] - mean[:, 0]).norm(dim=2) * pair_ok
        cnt = pair_ok.sum(dim=0)
        C = (pair.sum(dim=0) / cnt.clamp(min=1)).cpu().numpy()
        valid = (cnt > 0).to(torch.uint8).cpu().numpy()
        p = np.maximum(P_MIN, C / C.max() if C.max() > 0 else 0.0 * C)
    res = [C, valid, adv, active, p, None, None, None]
    return res + [None] * 4 if case["label"] else res


def _exact_update(case, seed):
    w, grads, m, v = _update_inputs(case, seed)
    norm = math.sqrt(sum(float(g.double().square().sum()) for g in grads))
    scale = min(1.0, 2.0 / (norm + 1e-6))
    b1, b2, lr, eps, t = 0.9, 0.999, 1e-5, 1e-8, 100
    W, M, S = [], [], []
    for wi, gi, mi, vi in zip(w, grads, m, v):
        g = gi.double() * scale
        M.append(b1 * mi.double() + (1 - b1) * g)
        S.append(b2 * vi.double() + (1 - b2) * g * g)
        W.append(wi.double() - lr * (M[-1] / (1 - b1 ** t)) / ((S[-1] / (1 - b2 ** t)).sqrt() + eps))
    out = [np.array([norm]), *W, *M, *S]
    if case["bf16"]:
        out += W
    if case["pack"]:
        out.append(None)            # the layout of the packed weights is the library's own
    return out


def _exact_step(case, seed):
    inp = _step_inputs(case, seed)
    A, d, ff, V, nk, T = case["A"], case["d"], case["ff"], case["V"], inp["n_kept_host"], inp["T"]
    if inp["capacity"] * A > 60000:
        return None                 # would take more than 20 seconds
    cap = inp["capacity"] * A
    w = {k: inp[k].double() for k in WEIGHTS}
    chunk = _to_gpu(inp["kept_host"])
    rows = (chunk[:, None] * A + torch.arange(A, device="cuda")[None, :]).reshape(-1)
    tok = inp["tokens"][rows].long().clamp(max=V - 1)
    adv = inp["adv"].double()[chunk // case["N"]].repeat_interleave(A)
    old = inp["logp_old"].double()[rows]
    M = rows.shape[0]
    scale = 1.0 / M if case["token_mean"] else 1.0 / T
    z64 = lambda shape: torch.zeros(shape, dtype=torch.float64, device="cuda")
    logp, ent = z64(cap), z64(M)
    block = A * max(1, 8192 // A)
    for r0 in range(0, M, block):
        x = inp["hidden"][rows[r0:r0 + block]].double()
        a = torch.nn.functional.silu(x @ w["Wg"]) * (x @ w["Wu"])
        lsm = torch.log_softmax((a @ w["Wd"]) @ w["Wo"], dim=1)
        logp[r0:r0 + x.shape[0]] = lsm.gather(1, tok[r0:r0 + block, None])[:, 0]
        ent[r0:r0 + x.shape[0]] = -(lsm.exp() * lsm).sum(dim=1)
    if not case["grads"]:
        return dict(logp=logp)
    delta = logp[:M] - old
    if case["chunk_ratio"]:
        delta = delta.view(-1, A).sum(dim=1).repeat_interleave(A)
    ratio = delta.exp()
    flows = torch.where(adv >= 0, ratio <= 1 + EPS_HIGH, ratio >= 1 - EPS_LOW)
    term = torch.minimum(ratio * adv, ratio.clamp(1 - EPS_LOW, 1 + EPS_HIGH) * adv)
    if case["chunk_ratio"]:
        term = term / A
    coef = torch.where(flows, -scale * ratio * adv, torch.zeros_like(adv))
    loss = -scale * term.sum() - case["entropy"] * scale * ent.sum()
    dW = {k: z64(w[k].shape) for k in WEIGHTS}
    dX = z64((cap, d))
    for r0 in range(0, M, block):
        x = inp["hidden"][rows[r0:r0 + block]].double()
        r1 = r0 + x.shape[0]
        u, v = x @ w["Wg"], x @ w["Wu"]
        sg = torch.sigmoid(u)
        a = u * sg * v
        y = a @ w["Wd"]
        lsm = torch.log_softmax(y @ w["Wo"], dim=1)
        pr = lsm.exp()
        dz = -coef[r0:r1, None] * pr
        dz.scatter_add_(1, tok[r0:r1, None], coef[r0:r1, None])
        if case["entropy"] != 0.0:
            dz += case["entropy"] * scale * pr * (lsm + ent[r0:r1, None])
        dW["Wo"] += y.T @ dz
        dy = dz @ w["Wo"].T
        dW["Wd"] += a.T @ dy
        da = dy @ w["Wd"].T
        du, dv = da * v * sg * (1 + u * (1 - sg)), da * u * sg
        dW["Wg"] += x.T @ du
        dW["Wu"] += x.T @ dv
        dX[r0:r1] = du @ w["Wg"].T + dv @ w["Wu"].T
    # the extended entry point reports the entropy as a fifth statistic, the plain one leaves it zero
    extended = any(case[k] for k in ("token_mean", "entropy", "chunk_ratio", "composed", "packed", "sumsq"))
    stats = torch.stack([1.0 - flows.double().mean(), ratio.mean(), (old - logp[:M]).mean(),
                         torch.tensor(float(M), dtype=torch.float64, device="cuda"), ent.mean() * float(extended)])
    out = dict(loss=loss.reshape(1), logp=logp, stats=stats)
    out.update({"d" + k: dW[k] for k in WEIGHTS})
    out["dX"] = dX
    if case["sumsq"]:
        out["grad_sumsq"] = sum(g.square().sum() for g in dW.values()).reshape(1)
    return out
