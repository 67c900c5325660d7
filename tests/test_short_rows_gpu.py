"""Verification, diagnostics and greedy verification of rows of 7 to 32 tiles, which are cut into up to four slices where there are few of
them and the workspace has svip_workspace_bytes: against the same calls with one slice per row.  Comparisons are exact; probabilities
and divergences differ by the order of fp32 and fp64 partial sums, logsumexps by 2^-22 of themselves at most, which is 1e-5 of a
probability at most for logsumexps below 40."""
import pytest
import torch

pytestmark = pytest.mark.gpu

BF, F16, F32 = torch.bfloat16, torch.float16, torch.float32
CASES = [(BF, 3, 5, 7 * 2048 - 3), (BF, 3, 5, 8 * 2048), (F16, 2, 7, 15 * 2048 + 1), (F32, 5, 4, 16 * 1024 - 5), (BF, 9, 6, 31 * 2048 + 9),
         (F32, 2, 3, 32 * 1024), (BF, 40, 5, 11 * 2048), (BF, 90, 5, 11 * 2048)]


@pytest.mark.parametrize("dtype,B,k,V", CASES)
@pytest.mark.parametrize("lse", [True, False])
def test_slices_of_short_rows(svip, dtype, B, k, V, lse):
    g = torch.Generator(device="cuda").manual_seed(V + B)
    per16 = 4 if dtype == F32 else 8
    stride = -(-V // per16) * per16
    draft = torch.empty(B, k, stride, dtype=dtype, device="cuda")[:, :, :V]
    target = torch.empty(B, k + 1, stride, dtype=dtype, device="cuda")[:, :, :V]
    z = torch.randn(B, k + 1, V, device="cuda", generator=g) * 4
    draft.copy_(z[:, :k])
    target.copy_(z + torch.randn(z.shape, device="cuda", generator=g))
    tokens = draft.float().argmax(-1).int()
    draft_len = torch.randint(0, k + 1, (B,), device="cuda", generator=g, dtype=torch.int32)
    draft_lse = torch.logsumexp(draft.double(), -1) if lse else None
    ua, ur = torch.rand(B, k, device="cuda", generator=g), torch.rand(B, device="cuda", generator=g)
    got = []
    try:
        for slices, exact in ((1, False), (0, False), (0, True)):          # exact: a workspace with no room for finer slices
            svip.bench_set_tuning(stats_slices=slices, pair_slices=slices)
            need = max(svip.workspace_needed(call, dtype, B, k, V) for call in ((1, 3, 4) if lse else (2, 3, 5)))
            ws = torch.zeros(need, dtype=torch.uint8, device="cuda") if exact else svip.new_workspace(B, k, V)
            o = {n: torch.full((B,), -7, dtype=torch.int32, device="cuda") for n in ("nacc", "next", "gacc", "gnext")}
            prob, stats = torch.zeros(B, k, device="cuda"), torch.zeros(B, k, svip.PAIR_NSTAT, device="cuda")
            svip.verify(target, draft, temperature=1.0, draft_tokens=tokens, draft_len=draft_len, draft_lse=draft_lse, u_accept=ua,
                        u_resample=ur, n_accepted_out=o["nacc"], next_token_out=o["next"], accept_prob_out=prob, workspace=ws)
            svip.verify_greedy(target, draft_tokens=tokens, draft_len=draft_len, n_accepted_out=o["gacc"], next_token_out=o["gnext"],
                               workspace=ws)
            svip.pair_stats(target, draft, temperature=1.0, draft_len=draft_len, c=0.18, stats_out=stats, workspace=ws, draft_lse=draft_lse)
            torch.cuda.synchronize()
            got.append((o, prob, stats[:, :, :4].nan_to_num(-1.0)))
    finally:
        svip.bench_set_tuning()
    for other in got[1:]:
        for n in got[0][0]:
            assert torch.equal(got[0][0][n], other[0][n]), n
        assert (got[0][1] - other[1]).abs().max() <= 1e-5
        assert ((got[0][2] - other[2]).abs() <= 1e-5 * got[0][2].abs().clamp_min(1.0)).all()


@pytest.mark.parametrize("dtype,B,k,V", [CASES[0], CASES[2], CASES[3], CASES[6], (BF, 2, 9, 25 * 2048 - 1)])
@pytest.mark.parametrize("lse", [True, False])
def test_results_by_workspace_and_against_64_bits(svip, dtype, B, k, V, lse):
    """The same bits in all workspaces of svip_workspace_bytes and more, and in all smaller ones; both within 1e-5 of probabilities and
    divergences in 64 bits."""
    g = torch.Generator(device="cuda").manual_seed(V)
    per16 = 4 if dtype == F32 else 8
    stride = -(-V // per16) * per16
    draft = torch.empty(B, k, stride, dtype=dtype, device="cuda")[:, :, :V]
    target = torch.empty(B, k + 1, stride, dtype=dtype, device="cuda")[:, :, :V]
    z = torch.randn(B, k + 1, V, device="cuda", generator=g) * 4
    draft.copy_(z[:, :k])
    target.copy_(z + torch.randn(z.shape, device="cuda", generator=g))
    tokens = draft.float().argmax(-1).int()
    draft_len = torch.full((B,), k, dtype=torch.int32, device="cuda")
    draft_lse = torch.logsumexp(draft.double(), -1) if lse else None
    ua, ur = torch.rand(B, k, device="cuda", generator=g), torch.rand(B, device="cuda", generator=g)
    least = max(svip.workspace_needed(call, dtype, B, k, V) for call in ((1, 4) if lse else (2, 5)))
    enough = svip.workspace_bytes(B, k, V)
    got = {}
    for size in (least, enough - 256, enough, enough + 4096):
        ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
        o = [torch.zeros(B, dtype=torch.int32, device="cuda") for _ in range(2)]
        prob, stats = torch.zeros(B, k, device="cuda"), torch.zeros(B, k, svip.PAIR_NSTAT, device="cuda")
        svip.verify(target, draft, temperature=1.0, draft_tokens=tokens, draft_len=draft_len, draft_lse=draft_lse, u_accept=ua, u_resample=ur,
                    n_accepted_out=o[0], next_token_out=o[1], accept_prob_out=prob, workspace=ws)
        svip.pair_stats(target, draft, temperature=1.0, draft_len=draft_len, c=0.18, stats_out=stats, workspace=ws, draft_lse=draft_lse)
        torch.cuda.synchronize()
        got[size] = (*o, prob, stats)
    for a, b in ((least, enough - 256), (enough, enough + 4096)):
        for x, y in zip(got[a], got[b]):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32))
    lp, lq = torch.log_softmax(target[:, :k].double(), -1), torch.log_softmax(draft.double(), -1)
    ratio = (lp - lq).gather(-1, tokens.long()[..., None])[..., 0].exp().clamp(max=1.0)
    q = lq.exp()
    kl, hq = (q * (lq - lp)).sum(-1), -(q * lq).sum(-1)
    want = torch.stack([torch.minimum(lp.exp(), q).sum(-1), kl, kl + hq, hq], -1)
    for size in (least, enough):
        assert (got[size][2] - ratio).abs().max() <= 1e-5
        assert ((got[size][3][:, :, :4] - want).abs() <= 1e-5 * want.abs().clamp_min(1.0)).all()


@pytest.mark.parametrize("dtype", [BF, F16, F32])
@pytest.mark.parametrize("tiles", [7, 8, 15, 16, 23, 31])
@pytest.mark.parametrize("lse", [True, False])
def test_rows_without_a_distribution_have_no_token(svip, dtype, tiles, lse):
    """A logit of +inf in any slice of a row that is cut finer: the same as with the longer slices, and where those are one per row no
    correction or bonus token (-1) and no rejection at that position; its neighbours are unaffected."""
    per16 = 4 if dtype == F32 else 8
    B, k, V = 6, 2, tiles * 256 * per16 - 3
    g = torch.Generator(device="cuda").manual_seed(tiles)
    stride = -(-V // per16) * per16
    draft = torch.empty(B, k, stride, dtype=dtype, device="cuda")[:, :, :V]
    target = torch.empty(B, k + 1, stride, dtype=dtype, device="cuda")[:, :, :V]
    z = torch.randn(B, k + 1, V, device="cuda", generator=g) * 4
    draft.copy_(z[:, :k])
    target.copy_(z + torch.randn(z.shape, device="cuda", generator=g))
    for b, at in enumerate((0, V // 4, V // 2, V - 1)):                    # sequences 4 and 5 have none
        target[b, 0, at] = float("inf")
    tokens = draft.float().argmax(-1).int()
    draft_len = torch.tensor([0, 0, 0, 0, 0, 2], dtype=torch.int32, device="cuda")
    for first in (0, 1):                       # the row is the bonus row, then the first position's target row
        draft_len[:5] = first
        results = []
        for size in (svip.workspace_bytes(B, k, V), max(svip.workspace_needed(c, dtype, B, k, V) for c in (1, 2))):
            ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
            nacc, nxt = (torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
            svip.verify(target, draft, temperature=1.0, draft_tokens=tokens, draft_len=draft_len,
                        draft_lse=torch.logsumexp(draft.double(), -1) if lse else None, u_accept=torch.full((B, k), 0.999, device="cuda"),
                        u_resample=torch.full((B,), 0.4, device="cuda"), n_accepted_out=nacc, next_token_out=nxt, accept_prob_out=None,
                        workspace=ws)
            torch.cuda.synchronize()
            results.append((nacc, nxt))
        for a, b in zip(*results):
            assert torch.equal(a, b) and (a[4:] >= 0).all()
        if tiles < 16:
            assert (results[0][0][:4] == first).all() and (first == 1 or (results[0][1][:4] == -1).all())
