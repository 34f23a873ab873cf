"""The fp32 actor step where its operands in blocks and as three bf16 matrices can go wrong: sizes at the edges of the padding and of the
tiles, the lines between its two routes, magnitudes at the ends of the fp32 range, values that are no numbers, and sums of one sign."""
import numpy as np
import pytest
import torch

from paper_2605_16154_amd import binding
from test_gpu_actor import CONFIGS, GRADS, check, condition_logp_old, make_problem, pcm, run_both  # noqa: F401

pytestmark = pytest.mark.gpu
TOL = 1e-5     # the accuracy that the fp32 path states


def problem(d, ff, V, A, n_kept, seed=5):
    cfg = CONFIGS["cfg1"].with_(n_groups=1, G=4, N=max(4, -(-n_kept // 3)), K=2, B=4, d=d, ff=ff, V=V, L=1, D=A, seed=seed)
    kept = np.arange(0, cfg.T * cfg.N)[:n_kept]
    # logits of order one, for which TOL is stated: their error, relative to the largest, is that of the ratios
    pr = make_problem(cfg, wstd=min(0.2, 1.2 / np.sqrt(d), 2.5 / np.sqrt(ff)), margin=1e-3, kept=kept, old_rel=0.2)
    pr["adv"] = np.where(np.arange(cfg.T) % 2 == 0, 0.8, -1.2)
    return pr


@pytest.mark.parametrize("composed", [False, True])
@pytest.mark.parametrize("d,ff,V,A,n_kept,max_kept", [
    (1, 1, 2, 1, 1, 1),               # one product per value
    (64, 128, 128, 1, 256, 256),      # whole steps, whole units of padding, one whole row tile
    (65, 129, 129, 1, 257, 300),      # one beyond each of them
    (63, 127, 127, 3, 85, 86),        # one before; rows unaligned to 16 bytes; 255 rows
    (130, 384, 384, 5, 103, 110),     # three units of padding: a 256-wide tile reaches beyond them
    (257, 640, 513, 4, 63, 64),       # V of five units; 252 rows
    (96, 2560, 1024, 8, 20, 70),      # the widest V; row tiles of the buffer without a live row
    (700, 300, 101, 15, 90, 90),      # six row tiles
])
def test_f32_sizes(pcm, d, ff, V, A, n_kept, max_kept, composed):   # noqa: F811
    """TOL holds at these sizes as at any: sums of at most 2560 terms in fp32."""
    pr = problem(d, ff, V, A, n_kept)
    for variants in ({}, dict(entropy_coef=1e-3, token_mean=True)):
        ref, got = run_both(pcm, pr, max_kept=max_kept, composed_head=composed, variants=variants, scale=1.0 if variants else None)
        check(ref, got, TOL, len(ref["rows"]))
        assert not got["dX"][len(ref["rows"]):].any()          # rows of the buffer behind the kept ones
    _, fwd = run_both(pcm, pr, max_kept=max_kept, composed_head=composed, want_grads=False, want_dX=False, scale=1.0 if variants else None,
                      variants=variants)
    n = len(ref["rows"])
    assert np.array_equal(fwd["logp"][:n], got["logp"][:n])
    _, only = run_both(pcm, pr, max_kept=max_kept, composed_head=composed, want_grads=False, want_dX=True, scale=1.0 if variants else None,
                       variants=variants)
    assert np.array_equal(only["dX"], got["dX"])


@pytest.mark.parametrize("power", [60, 80])
def test_f32_scaled_operands_give_the_same_bits(pcm, power):   # noqa: F811
    """Rows times 2^p and gate and up weights over 2^p: every product and sum scales exactly, parts of operands included
    (the smallest, 2^-16 of the smallest weight, is a normal bf16 value: checked)."""
    pr = problem(96, 160, 64, 4, 40)
    assert min(np.abs(pr["W"][k]).min() for k in ("Wg", "Wu")) * 2.0 ** (-power - 16) > 2.0 ** -125
    f = 2.0 ** power
    sc = dict(pr, hidden=(pr["hidden"].astype(np.float32) * np.float32(f)), W=dict(pr["W"], Wg=pr["W"]["Wg"].astype(np.float32) / np.float32(f),
                                                                                   Wu=pr["W"]["Wu"].astype(np.float32) / np.float32(f)))
    base = dict(pr, hidden=pr["hidden"].astype(np.float32), W={k: v.astype(np.float32) for k, v in pr["W"].items()})
    _, want = run_both(pcm, base)
    _, got = run_both(pcm, sc)
    for k in ("loss", "logp", "dWd", "dWo"):
        assert np.array_equal(got[k], want[k]), k
    for k in ("dWg", "dWu"):
        assert np.array_equal(got[k] / np.float32(f), want[k]), k
    assert np.array_equal(got["dX"] * np.float32(f), want["dX"])


def test_f32_largest_value(pcm):   # noqa: F811
    """The largest fp32 value splits without overflow: 2^128 (1 - 2^-24) times a weight of 2^-126 is 4 (1 - 2^-24)."""
    pr = problem(64, 96, 32, 4, 20)
    hidden, W = pr["hidden"].astype(np.float32), {k: v.astype(np.float32) for k, v in pr["W"].items()}
    hidden[:, 0] = np.finfo(np.float32).max
    W["Wg"][0] = W["Wu"][0] = np.float32(2.0 ** -126)
    ref, got = run_both(pcm, dict(pr, hidden=hidden, W=W), want_grads=False, want_dX=False)
    n = len(ref["rows"])
    assert np.isfinite(got["logp"][:n]).all()
    assert np.abs(got["logp"][:n] - ref["logp"]).max() <= TOL * np.abs(ref["logp"]).max()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_f32_rows_that_are_no_numbers_stay_alone(pcm, value):   # noqa: F811
    """A row with an infinity or a NaN has NaN for its log-probability; every other row is what it is without."""
    pr = problem(70, 90, 33, 4, 80)
    hidden = pr["hidden"].astype(np.float32)
    _, want = run_both(pcm, dict(pr, hidden=hidden), want_grads=False, want_dX=False)
    bad = hidden.copy()
    bad[17, 3] = value
    _, got = run_both(pcm, dict(pr, hidden=bad), want_grads=False, want_dX=False)
    others = np.arange(len(want["logp"])) != 17
    assert np.isnan(got["logp"][17]) and np.array_equal(got["logp"][others], want["logp"][others])


@pytest.mark.parametrize("composed", [False, True])
@pytest.mark.parametrize("d,ff,A,n_kept,max_kept", [
    (64, 128, 16, 176, 176),          # 2816 rows: the last as they are, 22 x 2^20 values of a row and the head
    (64, 128, 16, 177, 177),          # and the first in blocks (composed: as they are)
    (64, 80, 16, 2048, 2048),         # 32,768 rows: the last of a narrow head in blocks
    (64, 80, 16, 2049, 2049),         # and the first as they are
    (128, 288, 4, 312, 312),          # 1248 rows: composed as they are, 44 x 2^20 values of a row and the head at most
    (128, 288, 4, 313, 313),          # and in blocks
    (128, 289, 4, 20, 40),            # a head of more than 36 x 1024 values: in blocks whatever the rows
    (64, 129, 4, 20, 40),             # more than 8 x 1024
    (64, 64, 4, 20, 40),              # 4 x 1024: as they are
    (65, 64, 4, 20, 40),              # a few more, and few rows: as they are
])
def test_f32_routes(pcm, d, ff, A, n_kept, max_kept, composed):   # noqa: F811
    pr = problem(d, ff, 64, A, n_kept)
    for variants in ({}, dict(chunk_ratio=True, entropy_coef=1e-3)):
        # per-chunk ratio: the log-ratio of a chunk is a sum over its rows
        ref, got = run_both(pcm, pr, max_kept=max_kept, composed_head=composed, variants=variants)
        check(ref, got, 5 * TOL if variants else TOL, len(ref["rows"]), n_stats=5 if variants else 4)
        assert not got["dX"][len(ref["rows"]):].any()


@pytest.mark.parametrize("composed", [False, True])
@pytest.mark.parametrize("grads,least", [(True, 11409920), (False, 4590080)])
def test_f32_least_workspace(pcm, monkeypatch, grads, least, composed):   # noqa: F811
    """An fp32 call takes the bytes that every call of its shape took before operands went into blocks (720 rows of 192 -> 320 -> 128): the
    operands then stay as they are.  The forward pass has the same bits either way."""
    pr = problem(192, 320, 128, 8, 85)
    kw = dict(max_kept=90, composed_head=composed, want_grads=grads, want_dX=grads)
    _, whole = run_both(pcm, pr, **kw)
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    taken = []
    monkeypatch.setattr(binding, "_take_workspace", lambda need, dev, stream: taken.append(need) or ws)
    monkeypatch.setattr(binding, "_give_workspace", lambda *a: None)
    ref, got = run_both(pcm, pr, **kw)
    n = len(ref["rows"])
    assert taken[0] > least if grads else taken[0] >= least
    assert np.array_equal(got["loss"], whole["loss"]) and np.array_equal(got["logp"][:n], whole["logp"][:n])
    if grads:
        check(ref, got, TOL, n)
        assert not got["dX"][n:].any()
    ws = torch.empty(least - 256, dtype=torch.uint8, device="cuda")
    with pytest.raises(binding.PcmError, match="workspace"):
        run_both(pcm, pr, **kw)


def one_sign_problem(d, ff, V, A, n_kept, seed):
    """Weight gradients whose terms nearly all have one sign."""
    rng = np.random.default_rng(seed)
    f32 = lambda x: x.astype(np.float32).astype(np.float64)
    cfg = CONFIGS["cfg1"].with_(n_groups=1, G=4, N=n_kept, K=2, B=4, d=d, ff=ff, V=V, L=1, D=A, seed=seed)
    rows = cfg.T * cfg.N * A
    positive = lambda n, m, scale: f32((np.abs(rng.normal(size=(n, m))) + 0.5) * scale)
    hidden = positive(rows, d, 1.0)
    W = dict(Wg=positive(d, ff, 1.0 / d), Wu=positive(d, ff, 1.0 / d), Wd=positive(ff, d, 1.0 / ff), Wo=f32(rng.normal(size=(d, V)) * 0.2 / np.sqrt(d)))
    W["Wo"][:, 0] = f32(np.abs(rng.normal(size=d)) / d + 2.0 / d)             # every token is bin 0, whose logit every row raises
    x = hidden[:n_kept * A]
    u, v = x @ W["Wg"], x @ W["Wu"]
    z = (u / (1 + np.exp(-u)) * v) @ W["Wd"] @ W["Wo"]
    logp_old = np.full(rows, -5.5, np.float32)
    logp_old[:n_kept * A] = z[:, 0] - z.max(1) - np.log(np.exp(z - z.max(1, keepdims=True)).sum(1)) - 0.05    # ratios of 1.05: nothing is cut
    return dict(cfg=cfg, W=W, hidden=hidden, tokens=np.zeros(rows, np.uint8), logp_old=logp_old, adv=np.ones(cfg.T), kept=np.arange(n_kept))


@pytest.mark.parametrize("d,ff,V,A,n_kept,composed,least", [(256, 1024, 256, 56, 96, False, 129398272), (300, 700, 256, 56, 48, False, 71195648),
                                                            (473, 333, 512, 56, 96, True, 104272128)])
def test_f32_sums_of_one_sign(pcm, monkeypatch, d, ff, V, A, n_kept, composed, least):   # noqa: F811
    """Where all terms of a sum have one sign its roundings grow with it, most in long chains of additions: with operands in blocks the error
    against 64 bits is no larger than with operands as they are (`least` bytes of workspace), root mean square over four inputs; 1.05 for what
    the two have in common, the error of the ratios, and four inputs leave open."""
    error = {False: {k: [] for k in GRADS}, True: {k: [] for k in GRADS}}
    for seed in range(4):
        pr = one_sign_problem(d, ff, V, A, n_kept, seed)
        for direct in (False, True):
            with monkeypatch.context() as m:
                if direct:
                    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
                    m.setattr(binding, "_take_workspace", lambda need, dev, stream: ws)
                    m.setattr(binding, "_give_workspace", lambda *a: None)
                ref, got = run_both(pcm, pr, composed_head=composed)
            for k in GRADS:
                error[direct][k].append(np.linalg.norm(got[k] - ref[k]) / np.linalg.norm(ref[k]))
    rms = {route: {k: float(np.sqrt(np.mean(np.square(v)))) for k, v in e.items()} for route, e in error.items()}
    print(rms)
    for k in GRADS:
        assert rms[False][k] <= 1.05 * rms[True][k], (k, rms)
