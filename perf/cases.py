"""The work that a user of this library has it do, as timed cases.

A serving loop calls draft_step once per draft position and verify once per round (Algorithm 1), eagerly or
replayed from a HIP graph it captured over its static logit buffers; greedy decoding uses the greedy forms of
both; truncated sampling filters the rows with warp_logits first; pair_stats and Loop serve the analysis of
draft-length policies.  The sizes are those of this repository's workloads (svip_inputs.py, bench.py): batches
of 1 to 256, vocabularies of 32000, 128256 and 151936, 4 to 64 draft positions, fp32 and bf16 logits, and
between them odd vocabularies and fp16.

Logits are heavy-tailed like those of a language model: N(0, s^2) over the vocabulary with s of a row between
4 and 6.5, which puts the mass on a handful to some hundreds of tokens and the entropy between about 0.3 and
4 nats (the span the paper reports for accepted and rejected drafts).  Target rows are the draft rows plus
noise, so that most but not all drafts are accepted.
"""
import math

import torch

import paper_2411_18462_amd as svip

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
SIZE = {"f32": 4, "bf16": 2, "f16": 2}
H_OFF = 4.0                # above the square root of every row's entropy: all k positions are drafted


def listed():
    return [
        # one user, a small vocabulary, the calls made one by one: latency and launches are everything
        dict(name="round_one_user", kind="round", B=1, V=32000, k=8, dtype="f32", T=1.0, h=H_OFF),
        # a small server with a fixed draft length of five, eager calls on a large vocabulary
        dict(name="round_small_server", kind="round", B=8, V=128256, k=5, dtype="bf16", T=1.0, h=H_OFF),
        # the drafting phase of the benchmark's round, replayed from a graph
        dict(name="draft_64", kind="draft", B=64, V=128256, k=16, dtype="bf16", T=1.0, h=H_OFF),
        # the drafting phase of a large batch, another temperature
        dict(name="draft_256", kind="draft", B=256, V=151936, k=4, dtype="bf16", T=0.7, h=H_OFF),
        # fp32 logits of a middling batch
        dict(name="draft_16_f32", kind="draft", B=16, V=32000, k=16, dtype="f32", T=1.0, h=H_OFF),
        # verification of the benchmark's round, every position drafted
        dict(name="verify_64", kind="verify", B=64, V=128256, k=16, dtype="bf16", T=1.0, ragged=False, lse=True),
        # few sequences with long drafts of different lengths
        dict(name="verify_long_drafts", kind="verify", B=8, V=151936, k=64, dtype="bf16", T=1.0, ragged=True, lse=True),
        # a drafter that kept no logsumexps, fp16 logits, a vocabulary that fills no whole tile
        dict(name="verify_recompute_f16", kind="verify", B=32, V=50257, k=8, dtype="f16", T=0.8, ragged=True, lse=False),
        # greedy decoding (reasoning models), the whole round from a graph
        dict(name="greedy_64", kind="greedy", B=64, V=128256, k=16, dtype="bf16", T=1.0, h=H_OFF),
        # acceptance analysis of a batch of rounds
        dict(name="pair_stats_64", kind="pair", B=64, V=128256, k=16, dtype="bf16", T=1.0, ragged=True, lse=True),
        # nucleus filtering of a round's target rows
        dict(name="nucleus_round", kind="warp", B=64, V=128256, k=17, dtype="bf16", T=1.0, top_k=0, top_p=0.9),
        # a whole generation of a batch of eight under the entropy rule, greedy, over logit traces
        dict(name="loop_svip", kind="loop", B=8, V=151936, k=40, dtype="bf16", T=1.0, h=1.5, max_new=48),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["round", "draft", "verify", "greedy", "pair", "warp", "loop"])
    dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
    V = rng.choice([_log_uniform(rng, 8000, 152064), rng.choice([32000, 50257, 128256, 151936])])
    T = rng.choice([1.0, 1.0, 0.7, round(rng.uniform(0.5, 1.5), 2)])
    c = dict(kind=kind, dtype=dtype, V=V, T=T)
    if kind == "round":
        c.update(B=_log_uniform(rng, 1, 24), k=rng.randint(1, 12), h=rng.choice([H_OFF, 1.5]))
    elif kind == "loop":
        c.update(B=rng.randint(1, 12), k=rng.randint(4, 40), h=rng.choice([1.2, 1.5, 1.8]), max_new=rng.randint(8, 40))
    else:
        c.update(B=_log_uniform(rng, 1, 256), k=_log_uniform(rng, 1, 64))
    if kind in ("draft", "greedy"):
        c["h"] = H_OFF
    if kind == "pair":
        c["T"] = max(T, 1.0)
    if kind in ("verify", "pair"):
        c.update(ragged=rng.random() < 0.6, lse=rng.random() < 0.7)
    if kind == "warp":
        c["top_k"], c["top_p"] = rng.choice([(0, 0.9), (0, 0.95), (50, 1.0), (50, 0.9), (rng.randint(1, 1024), 0.8)])
    rows = {"loop": lambda: 2 * (c["max_new"] + c["k"] + 1)}.get(kind, lambda: 2 * c["k"] + 1)
    while c["B"] > 1 and c["B"] * rows() * V * SIZE[dtype] > 500e6:      # no larger than the largest listed case
        c["B"] = max(1, c["B"] // 2)
    return c


# ---- inputs -----------------------------------------------------------------------------------

def _row_stride(V, dtype):
    per16 = 16 // SIZE[dtype]
    return (V + per16 - 1) // per16 * per16         # rows start on 16-byte boundaries


def _empty_rows(B, n, V, dtype):
    return torch.empty(B, n, _row_stride(V, dtype), dtype=DTYPES[dtype], device="cuda")[:, :, :V]


def _logits(c, n_draft, n_target, g):
    """Draft rows [B, n_draft, V] and target rows [B, n_target, V], equal numbers or one more target row."""
    B, V, dt = c["B"], c["V"], c["dtype"]
    draft, target = _empty_rows(B, n_draft, V, dt), _empty_rows(B, n_target, V, dt)
    step = max(1, (1 << 27) // (n_target * V))
    for b in range(0, B, step):
        n = min(step, B - b)
        s = 4.0 + 2.5 * torch.rand(n, n_target, 1, device="cuda", generator=g)
        z = torch.randn(n, n_target, V, device="cuda", generator=g) * s
        draft[b:b + n] = z[:, :n_draft]
        z[:, :n_draft] = draft[b:b + n].float()
        target[b:b + n] = z + torch.randn(n, n_target, V, device="cuda", generator=g)
    return draft, target


def _draws(draft, T, g):
    """Tokens drawn from softmax(draft / T) and the rows' logsumexps in fp64, as a drafter would have them."""
    B, k, V = draft.shape
    tokens = torch.empty(B, k, dtype=torch.int32, device="cuda")
    lse = torch.empty(B, k, dtype=torch.float64, device="cuda")
    step = max(1, (1 << 26) // (k * V))
    for b in range(0, B, step):
        z = draft[b:b + step].float() / T
        lse[b:b + step] = torch.logsumexp(draft[b:b + step].double() / T, -1)
        z -= torch.log(-torch.log(torch.rand(z.shape, device="cuda", generator=g).clamp_(1e-12, 1 - 1e-7)))
        tokens[b:b + step] = z.argmax(-1).int()
    return tokens, lse


def _lengths(c, g):
    if not c.get("ragged"):
        return torch.full((c["B"],), c["k"], dtype=torch.int32, device="cuda")
    return torch.randint(1, c["k"] + 1, (c["B"],), device="cuda", generator=g, dtype=torch.int32)


def prepare(case, seed):
    c = dict(case)
    kind, B, V, k = c["kind"], c["B"], c["V"], c["k"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + B * 8191 + V * 31 + k)

    def full(value, *shape, dtype):
        return torch.full(shape, value, dtype=dtype, device="cuda")

    if kind == "loop":
        n = c["max_new"] + k + 1
        c["draft"], c["target"] = _logits(c, n, n, g)
        return c
    if kind == "warp":
        c["logits"], _ = _logits(c, k, k, g)
        c["out"] = _empty_rows(B, k, V, c["dtype"])
        c["kept"] = full(0, B * k, dtype=torch.int32)
        return c
    c["draft"], c["target"] = _logits(c, k, k + 1, g)
    c["ws"] = svip.new_workspace(B, k, V)
    if kind in ("verify", "pair"):
        c["tokens"], lse = _draws(c["draft"], c["T"], g)
        c["draft_lse"] = lse if c["lse"] else None
        c["draft_len"] = _lengths(c, g)
        if kind == "pair":
            c["stats"] = full(0.0, B, k, svip.PAIR_NSTAT, dtype=torch.float32)
            return c
        c["accept_prob"] = full(0.0, B, k, dtype=torch.float32)
    else:
        c["u_sample"] = torch.rand(B, k, device="cuda", generator=g)
        c["tokens"] = full(-1, B, k, dtype=torch.int32)
        c["draft_lse"] = full(0.0, B, k, dtype=torch.float64)
        c["entropy"] = full(0.0, B, k, dtype=torch.float32)
        c["q_tok"] = full(0.0, B, k, dtype=torch.float32)
        c["stop"] = full(0, B, dtype=torch.uint8)
        c["draft_len"] = full(0, B, dtype=torch.int32)
    c["u_accept"] = torch.rand(B, k, device="cuda", generator=g)
    c["u_resample"] = torch.rand(B, device="cuda", generator=g)
    c["n_accepted"] = full(-1, B, dtype=torch.int32)
    c["next_token"] = full(-1, B, dtype=torch.int32)
    if kind in ("draft", "greedy"):
        # a server with static logit buffers captures its calls once and replays them
        work = _drafting if kind == "draft" else _greedy_round
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            work(c)
        torch.cuda.current_stream().wait_stream(side)
        c["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(c["graph"]):
            work(c)
    return c


# ---- one pass ---------------------------------------------------------------------------------

def _drafting(s, greedy=False):
    for j in range(s["k"]):
        svip.draft_step(s["draft"][:, j], temperature=s["T"], h=s["h"], step_j=j, k_max=s["k"], greedy=greedy,
                        u_sample=None if greedy else s["u_sample"][:, j], stop_in=s["stop"] if j else None,
                        token_out=s["tokens"][:, j], entropy_out=s["entropy"][:, j], q_tok_out=s["q_tok"][:, j],
                        lse_out=s["draft_lse"][:, j], stop_out=s["stop"], draft_len_out=s["draft_len"],
                        workspace=s["ws"])


def _greedy_round(s):
    _drafting(s, greedy=True)
    svip.verify_greedy(s["target"], draft_tokens=s["tokens"], draft_len=s["draft_len"], n_accepted_out=s["n_accepted"],
                       next_token_out=s["next_token"], workspace=s["ws"])


def _verify(s):
    svip.verify(s["target"], s["draft"], temperature=s["T"], draft_tokens=s["tokens"], draft_len=s["draft_len"],
                draft_lse=s["draft_lse"], u_accept=s["u_accept"], u_resample=s["u_resample"],
                n_accepted_out=s["n_accepted"], next_token_out=s["next_token"], accept_prob_out=s.get("accept_prob"),
                workspace=s["ws"])


def run(s):
    kind = s["kind"]
    if kind == "warp":
        svip.warp_logits(s["logits"], temperature=s["T"], top_k=s["top_k"], top_p=s["top_p"], out=s["out"],
                         kept_out=s["kept"])
        return {"out": s["out"], "kept": s["kept"]}
    if kind == "pair":
        svip.pair_stats(s["target"], s["draft"], temperature=s["T"], draft_len=s["draft_len"], c=0.18,
                        stats_out=s["stats"], workspace=s["ws"], draft_lse=s["draft_lse"])
        return {"stats": s["stats"]}
    if kind == "loop":
        loop = svip.Loop(s["target"], s["draft"], temperature=s["T"], h=s["h"], gamma0=s["k"], gamma_max=s["k"],
                         max_new=s["max_new"], rounds=s["max_new"], greedy=True)
        loop.run()
        return {"state": loop.state, "tokens": loop.out_tokens}
    if kind == "verify":
        _verify(s)
        return {n: s[n] for n in ("n_accepted", "next_token", "accept_prob")}
    if kind in ("draft", "greedy"):
        s["graph"].replay()
    else:
        _drafting(s)
        _verify(s)
    drafted = {n: s[n] for n in ("tokens", "entropy", "q_tok", "draft_lse", "stop", "draft_len")}
    if kind == "draft":
        return drafted
    return dict(drafted, n_accepted=s["n_accepted"], next_token=s["next_token"])


# ---- what a pass cannot do without, and how far two correct ones are apart ------------------------

def work(case):
    c = case
    row, B, k = c["V"] * SIZE[c["dtype"]], c["B"], c["k"]
    mean_len = (k + 1) / 2 if c.get("ragged") else k
    kind = c["kind"]
    if kind == "draft":                 # every draft row once
        rows, ops = B * k, 6
    elif kind == "round":               # draft rows, then the target rows (rows of stopped sequences are not read)
        rows, ops = (B * (2 * k + 1) if c["h"] == H_OFF else B * 3), 5
    elif kind == "greedy":
        rows, ops = B * (2 * k + 1), 4
    elif kind == "verify":              # target rows of drafted positions, and draft rows: all or the rejected one
        rows, ops = B * (mean_len + 1 + (1 if c["lse"] else mean_len)), 4
    elif kind == "pair":                # both rows of every drafted position
        rows, ops = B * mean_len * 2, 8
    elif kind == "warp":                # read once, written once
        rows, ops = 2 * B * k, 3
    else:                               # one draft and one target row for every token produced
        rows, ops = B * c["max_new"] * 2, 4
    return {"bytes": rows * row, "flops": rows * c["V"] * ops}


def tolerance(case):
    """Measured against the same quantities in fp64: logsumexps 2e-8, entropies 6e-8 and probabilities 4e-8 relative
    (largest single difference 2e-7), divergences 2e-7.  A draw whose uniform lies within rounding of the edge between
    two tokens may take either: that moves one whole value, and one probability from one small cell to the next.
    Filtered logits are copies, greedy tokens comparisons."""
    kind = case["kind"]
    if kind in ("warp", "loop"):
        return "exact"
    if kind == "pair":        # entropies near zero stand in the denominator of one of the statistics
        return {"rel": 1e-5, "max": 1e-3}
    if kind == "verify":
        return {"rel": 4e-7, "max": 4e-6, "differ": 0.01}
    return {"rel": 1e-6, "max": 4e-5, "differ": 0.01}
