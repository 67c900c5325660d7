"""The launch of svip_verify that tests acceptance and draws the token: drafts longer than a wave, outputs that lie on inputs,
slices of every length, and rejections without residual mass.  Against the oracle (decision by decision, test_edges_gpu.py has
the vocabulary sizes) or against the same call in its usual form, which must agree bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_verify, Round

pytestmark = pytest.mark.gpu


def _case(B, k, V, dtype, seed, noise=0.8):
    g = torch.Generator().manual_seed(seed)
    draft = (3.0 * torch.randn(B, k, V, generator=g)).to(dtype)
    target = torch.cat([draft.float(), 3.0 * torch.randn(B, 1, V, generator=g)], 1)
    target = (target + noise * torch.randn(B, k + 1, V, generator=g)).to(dtype)
    u = torch.rand(3, B, k, generator=g)
    return draft, target, u[0], u[1], u[2][:, 0].contiguous()


@pytest.mark.parametrize("k", [1, 63, 64, 65, 130])
@pytest.mark.parametrize("lse", ["given", None])
def test_long_drafts(svip, k, lse):
    """Acceptance in passes of 64 positions; with little noise rejections lie in every pass."""
    B, V = 5, 2056
    print(f"verify draw k={k} lse={lse}", flush=True)
    draft, target, us, ua, ur = _case(B, k, V, torch.bfloat16, 3 * k, noise=0.02)
    r = Round(svip, draft, target, us, ua, ur, 1.0, 100.0)
    r.draft_all(chain=False)
    tokens = r.tokens.cpu().numpy().astype(np.int64)
    dl = np.array([k, max(k - 1, 0), k // 2, 0, min(k, 64)], np.int64)
    r.verify(tokens=r.tokens, draft_len=torch.from_numpy(dl).int().cuda(), lse=lse)
    check_verify(draft, target, 1.0, tokens, dl, ua, ur, r)


def _verify(svip, draft, target, tokens, dlen, lse, ua, ur, nacc, nxt, prob, **tuning):
    B, k, V = draft.shape
    ws = svip.new_workspace(B, k, V)
    try:
        svip.bench_set_tuning(**tuning)
        svip.verify(target, draft, temperature=1.0, draft_tokens=tokens, draft_len=dlen, draft_lse=lse, u_accept=ua, u_resample=ur,
                    n_accepted_out=nacc, next_token_out=nxt, accept_prob_out=prob, workspace=ws)
        torch.cuda.synchronize()
    finally:
        svip.bench_set_tuning()
    assert svip.workspace_flags(ws) == 0


@pytest.mark.parametrize("B,k,V,dtype", [(9, 16, 32000, torch.float32), (17, 70, 50257, torch.float16), (64, 3, 128256, torch.bfloat16)])
def test_outputs_on_inputs_and_slices_of_any_length(svip, B, k, V, dtype):
    """n_accepted_out may be draft_len and accept_prob_out may be u_accept; one, some and the most slices a row can have."""
    print(f"verify draw B={B} k={k} V={V} {dtype}", flush=True)
    mult = 4 if dtype == torch.float32 else 8
    Vp = (V + mult - 1) // mult * mult
    g = torch.Generator(device="cuda").manual_seed(B)
    draft = torch.empty(B, k, Vp, dtype=dtype, device="cuda")[:, :, :V]
    target = torch.empty(B, k + 1, Vp, dtype=dtype, device="cuda")[:, :, :V]
    draft.copy_(3.0 * torch.randn(B, k, V, device="cuda", generator=g))
    target.copy_(3.0 * torch.randn(B, k + 1, V, device="cuda", generator=g))
    target[:, :k] = draft + 0.2 * target[:, :k]
    ua, ur = torch.rand(B, k, device="cuda", generator=g), torch.rand(B, device="cuda", generator=g)
    tokens = torch.randint(0, V, (B, k), device="cuda", generator=g, dtype=torch.int32)
    tokens[:, : k // 2] = draft[:, : k // 2].argmax(-1).int()
    dlen = torch.randint(0, k + 1, (B,), device="cuda", generator=g, dtype=torch.int32)
    lse = torch.logsumexp(draft.double(), -1)

    def out():
        return (torch.full((B,), -5, dtype=torch.int32, device="cuda"), torch.full((B,), -5, dtype=torch.int32, device="cuda"),
                torch.full((B, k), -5.0, device="cuda"))
    n0, t0, p0 = out()
    _verify(svip, draft, target, tokens, dlen, lse, ua, ur, n0, t0, p0)
    inside = torch.arange(k, device="cuda")[None] < dlen[:, None]
    assert (p0[inside] >= 0).all() and (p0[~inside] == -5.0).all() and (t0 >= 0).all() and (n0 <= dlen).all()
    d1, u1 = dlen.clone(), ua.clone()
    _, t1, _ = out()
    _verify(svip, draft, target, tokens, d1, lse, u1, ur, d1, t1, u1)
    assert torch.equal(d1, n0) and torch.equal(t1, t0) and torch.equal(u1[inside], p0[inside])
    tiles = -(-(-(-V // mult)) // 256)
    for ns in sorted({1, 2, -(-tiles // 4), min(64, tiles)}):      # 1, 2: slices longer than four tiles where the row is
        n2, t2, p2 = out()
        _verify(svip, draft, target, tokens, dlen, lse, ua, ur, n2, t2, p2, resid_slices=ns)
        assert torch.equal(n2, n0) and torch.equal(p2, p0), ns
        # partial sums are rounded differently: a draw within rounding of a cell's edge may move to the next cell
        assert (t2 != t0).sum() <= 1 + B // 16, ns


@pytest.mark.parametrize("V,dtype", [(40, torch.float32), (5001, torch.bfloat16), (32000, torch.float16), (32005, torch.float32), (530001, torch.bfloat16)])
def test_rejection_without_residual_mass_draws_from_the_target(svip, V, dtype):
    """Logsumexps 1 too small make q = e p everywhere: a token is rejected with u >= 1 / e, and nothing of p is above q."""
    print(f"verify draw without mass V={V} {dtype}", flush=True)
    B, k = 24, 2
    mult = 4 if dtype == torch.float32 else 8
    Vp = (V + mult - 1) // mult * mult
    g = torch.Generator(device="cuda").manual_seed(V)
    draft = torch.empty(B, k, Vp, dtype=dtype, device="cuda")[:, :, :V]
    target = torch.empty(B, k + 1, Vp, dtype=dtype, device="cuda")[:, :, :V]
    target.copy_(2.0 * torch.randn(B, k + 1, V, device="cuda", generator=g))
    draft.copy_(target[:, :k])
    ua = torch.full((B, k), 0.2, device="cuda")
    ua[:, 1] = 0.9                                              # position 0 is accepted, position 1 is not
    ur = torch.rand(B, device="cuda", generator=g)
    tokens = draft.argmax(-1).int()
    dlen = torch.full((B,), k, dtype=torch.int32, device="cuda")
    lse = torch.logsumexp(draft.double(), -1) - 1.0
    nacc, nxt = torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty(B, dtype=torch.int32, device="cuda")
    _verify(svip, draft, target, tokens, dlen, lse, ua, ur, nacc, nxt, None)
    assert (nacc == 1).all()
    for b in range(B):
        p, _ = oracle.softmax_row(target[b, 1].double().cpu().numpy(), 1.0)
        c = np.concatenate([[0.0], np.cumsum(p)])
        t, u = int(nxt[b]), float(ur[b])
        assert p[t] > 0 and c[t] - 2e-6 <= u * c[-1] <= c[t + 1] + 2e-6, (b, t, u)


@pytest.mark.parametrize("k", [64, 70, 130])
@pytest.mark.parametrize("mass", [True, False])
def test_next_token_on_the_draft_lengths(svip, k, mass):
    """next_token_out may be draft_len, whether a draft has one pass of positions or several, and whether a rejection leaves
    residual mass or not (see test_rejection_without_residual_mass_draws_from_the_target)."""
    B, V = 9, 4104
    print(f"verify draw next token on draft_len k={k} mass={mass}", flush=True)
    draft, target, _, ua, ur = (x.cuda() for x in _case(B, k, V, torch.bfloat16, k, noise=0.05))
    if not mass:
        draft = target[:, :k].clone()
        ua[:] = 0.2
        ua[:, k // 2] = 0.9
    lse = torch.logsumexp(draft.double(), -1) - (0.0 if mass else 1.0)
    tokens = draft.argmax(-1).int()
    dlen = torch.tensor([k, k - 1, k // 2 + 1, 0, min(k, 64), 1, min(k, 65), k, k], dtype=torch.int32, device="cuda")

    def out():
        return torch.full((B,), -5, dtype=torch.int32, device="cuda"), torch.full((B, k), -5.0, device="cuda")
    (n0, p0), (n1, p1) = out(), out()
    t0, d1 = n0.clone(), dlen.clone()
    _verify(svip, draft, target, tokens, dlen, lse, ua, ur, n0, t0, p0)
    _verify(svip, draft, target, tokens, d1, lse, ua, ur, n1, d1, p1)         # checks the flags too
    assert torch.equal(n0, n1) and torch.equal(t0, d1) and torch.equal(p0, p1)


@pytest.mark.parametrize("k,at", [(64, 50), (70, 66), (200, 130), (200, 40)])
def test_flags_of_tokens_behind_the_first_rejection(svip, k, at):
    """A bad token is recorded if its position was tested: in the 64 positions of the first rejection, and behind them only
    where the accept probabilities are asked for."""
    B, V = 3, 1000
    draft, target, _, ua, ur = (x.cuda() for x in _case(B, k, V, torch.float32, k))
    tokens = draft.argmax(-1).int()
    ws = svip.new_workspace(B, k, V)
    target[:, 3] = target[:, 3].scatter(1, tokens[:, 3:4].long(), -float("inf"))         # position 3 at the latest is rejected
    tokens[1, at] = V + 7
    dlen = torch.full((B,), k, dtype=torch.int32, device="cuda")
    nacc, nxt = torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty(B, dtype=torch.int32, device="cuda")
    for prob in (None, torch.empty(B, k, device="cuda")):
        svip.verify(target, draft, temperature=1.0, draft_tokens=tokens, draft_len=dlen, draft_lse=torch.logsumexp(draft.double(), -1),
                    u_accept=ua, u_resample=ur, n_accepted_out=nacc, next_token_out=nxt, accept_prob_out=prob, workspace=ws)
        assert (nacc <= 3).all()
        seen = at < 64 or prob is not None
        assert svip.workspace_flags(ws) == (svip.FLAG_BAD_TOKEN if seen else 0), prob is not None


@pytest.mark.parametrize("B,more,V,dtype", [(2560, 2568, 8000, torch.float16), (304, 312, 40000, torch.bfloat16), (512, 520, 28672, torch.bfloat16)])
def test_acceptance_in_the_draws_launch_and_in_its_own(svip, B, more, V, dtype):
    """`B` sequences are the most whose acceptance test runs inside the residual pass (2560 workgroups of up to four slices a
    sequence, 1536 of more, 1024 of slices longer than four tiles): with eight more it has a launch of its own, and the same
    sequences get the same results."""
    k = 1
    print(f"verify draw in its own launch B={more} V={V} {dtype}", flush=True)
    draft, target, _, ua, ur = (x.cuda() for x in _case(more, k, V, dtype, V))
    lse, tokens = torch.logsumexp(draft.double(), -1), draft.argmax(-1).int()
    dlen = (torch.arange(more, device="cuda") % 2).int()
    full = [torch.full(s, -5, dtype=t, device="cuda") for s, t in (((more,), torch.int32), ((more,), torch.int32), ((more, k), torch.float32))]
    part = [x[:B].clone() for x in full]
    _verify(svip, draft, target, tokens, dlen, lse, ua, ur, *full)
    _verify(svip, draft[:B], target[:B], tokens[:B], dlen[:B], lse[:B], ua[:B], ur[:B], *part)
    for x, y in zip(full, part):
        assert torch.equal(x[:B], y)
    assert (full[0] >= 0).all() and (full[1] >= 0).all() and (full[0] == 0).any() and (full[0] == 1).any()
