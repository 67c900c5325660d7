"""Verification and diagnostics of rows masked with the type's lowest finite number (as torch.finfo(dtype).min, which many samplers write
instead of -inf) or with -inf, against the same quantities in 64 bits.  Such a logit has no weight next to any other, in
whatever part of the row it stands: whole threads, waves and slices may see nothing else.  Probabilities to 1e-5, as elsewhere; tokens
where the draw is not within 1e-6 of an edge between two."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

BF, F16, F32 = torch.bfloat16, torch.float16, torch.float32


def _masks(V, per, g):
    idx = torch.arange(V)
    return {"first third": idx < V // 3, "last two thirds": idx >= V // 3, "second quarter": (idx >= V // 4) & (idx < V // 2),
            "all but 20": ~torch.isin(idx, torch.randint(0, V, (20,), generator=g)),
            "nine of ten": torch.rand(V, generator=g) < 0.9, "all but a run": (idx < V // 2) | (idx >= V // 2 + 300),
            "most of the first tile": idx < 256 * per - 37}


@pytest.mark.parametrize("dtype", [BF, F32, F16])
@pytest.mark.parametrize("tiles", [1, 3, 10, 15, 16, 23, 25, 40])
@pytest.mark.parametrize("value", ["lowest", "-inf"])
def test_masked_rows_against_64_bits(svip, dtype, tiles, value):
    print(f"masked rows {dtype} tiles={tiles} {value}", flush=True)
    per = 4 if dtype == F32 else 8
    B, k, V = 6, 3, tiles * 256 * per - 5
    g = torch.Generator().manual_seed(tiles)
    n = torch.tensor([0, 1, 2, 3, 3, 2], dtype=torch.int32, device="cuda")
    u = torch.linspace(0.05, 0.95, B, device="cuda")
    base = torch.randn(B, k + 1, V, generator=g) * 4
    other = base + torch.randn(base.shape, generator=g)
    full = svip.workspace_bytes(B, k, V)
    least = max(svip.workspace_needed(call, dtype, B, k, V) for call in (1, 2, 4, 5))
    for name, mask in _masks(V, per, g).items():
        draft, target = (torch.empty(B, r, -(-V // per) * per, dtype=dtype, device="cuda")[:, :, :V] for r in (k, k + 1))
        for t, z in ((draft, base[:, :k]), (target, other)):
            z = z.to(dtype, copy=True)
            z[:, :, mask] = torch.finfo(dtype).min if value == "lowest" else -math.inf
            t.copy_(z)
        lp, lq = torch.log_softmax(target.double(), -1), torch.log_softmax(draft.double(), -1)
        tokens = lq.exp().float().view(B * k, V).multinomial(1).view(B, k).int()
        ratio = (lp[:, :k] - lq).gather(-1, tokens.long()[..., None])[..., 0].exp().clamp(max=1.0)
        beta = torch.minimum(lp[:, :k].exp(), lq.exp()).sum(-1)
        drafted = torch.arange(k, device="cuda")[None] < n[:, None]
        cdf = lp[torch.arange(B, device="cuda"), n.long()].exp().cumsum(-1)
        at = u.double()[:, None] * cdf[:, -1:]
        bonus, clear = (cdf <= at).sum(-1), (cdf - at).abs().amin(-1) > 1e-6
        for lse in (torch.logsumexp(draft.double(), -1), None):
            for size in (full, least):
                ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
                nacc, nxt = (torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
                prob, stats = torch.zeros(B, k, device="cuda"), torch.zeros(B, k, svip.PAIR_NSTAT, device="cuda")
                svip.verify(target, draft, temperature=1.0, draft_tokens=tokens, draft_len=n, draft_lse=lse,
                            u_accept=torch.zeros(B, k, device="cuda"), u_resample=u, n_accepted_out=nacc, next_token_out=nxt,
                            accept_prob_out=prob, workspace=ws)
                svip.pair_stats(target, draft, temperature=1.0, draft_len=n, c=0.18, stats_out=stats, workspace=ws, draft_lse=lse)
                torch.cuda.synchronize()
                assert ((prob - ratio).abs()[drafted] <= 1e-5).all(), (name, size)
                assert ((stats[..., 0] - beta).abs()[drafted] <= 1e-5).all(), (name, size)
                assert torch.equal(nacc, n) and (nxt[clear] == bonus[clear]).all(), (name, size)
