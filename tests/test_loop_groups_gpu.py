"""The decoding loop with several draft positions per launch against the loop that takes them one by one (which it still does
where a position alone fills the chip, and where an override asks for records of another size): state, tokens and log are the
same bit for bit.  64 records per row, the override used here, is what the rows of these shapes have anyway, so both sides
sum the same partial results."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _trace(B, L, V, dtype, seed, masked):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    per16 = 16 // torch.empty(0, dtype=dtype).element_size()
    stride = (V + per16 - 1) // per16 * per16
    out = []
    z = torch.randn(B, L, V, device="cuda", generator=g) * (2.0 + 4.0 * torch.rand(B, L, 1, device="cuda", generator=g))
    for noise in (0.0, 0.5):
        t = torch.empty(B, L, stride, dtype=dtype, device="cuda")[:, :, :V]
        t.copy_(z + noise * torch.randn(B, L, V, device="cuda", generator=g))
        if masked:
            t[:, ::3, : V // 2] = -math.inf                                     # whole tiles of masked logits
            t[:, 1::4, 5] = t[:, 1::4].amax(-1)                                 # ties for the maximum
            t[:, 2::5, V // 3:] = torch.finfo(dtype).min
        out.append(t)
    return out


def _loop(svip, draft, target, *, B, k, h, max_new, greedy, inc=0, dec=0, gamma0=None, chunk=None, T=1.0, one_by_one=False, seed=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 1)
    R = max_new
    u = {} if greedy else dict(u_sample=torch.rand(R, B, k, device="cuda", generator=g),
                               u_accept=torch.rand(R, B, k, device="cuda", generator=g),
                               u_resample=torch.rand(R, B, device="cuda", generator=g))
    try:
        if one_by_one:
            svip.bench_set_tuning(draft_slices=64)
        loop = svip.Loop(target, draft, temperature=T, h=h, gamma0=gamma0 or k, gamma_max=k, gamma_inc=inc, gamma_dec=dec,
                         max_new=max_new, rounds=R, greedy=greedy, check_every=4, **u)
        ran, running = [], 1
        while running and loop.next_round < R:
            n, running = loop.run(chunk)
            ran.append(n)
            if chunk:
                assert n <= chunk
    finally:
        svip.bench_set_tuning()
    assert running == 0 and loop.flags() == 0
    assert sum(ran) == int(loop.state[:, 3].max())
    n = sum(ran)
    return dict(ran=ran, running=running, state=loop.state.cpu(), out=loop.out_tokens.cpu(), log=loop.round_log.cpu()[:n])


@pytest.mark.parametrize("greedy", [True, False])
@pytest.mark.parametrize("B,k,V,dtype,policy,masked", [
    (1, 3, 8000, torch.bfloat16, "svip", False),          # one sequence: a whole draft per launch
    (7, 13, 32000, torch.float32, "svip", True),          # fewer rows than XCDs; a draft of several groups
    (9, 40, 50257, torch.float16, "svip", True),          # rows padded to 16; a vocabulary that fills no vector
    (12, 5, 128256, torch.bfloat16, "constant", False),
    (8, 70, 2049, torch.bfloat16, "heuristic", False),    # drafts longer than a wave; one logit in the second tile
    (33, 9, 32001, torch.float32, "svip", False),         # two positions per launch (greedy)
    (3, 1, 1000, torch.float32, "svip", False),           # drafts of one token, less than a tile
])
def test_groups_match_positions_one_by_one(svip, B, k, V, dtype, policy, masked, greedy):
    print(f"loop groups B={B} k={k} V={V} {dtype} {policy} greedy={greedy}", flush=True)
    max_new = 24
    draft, target = _trace(B, max_new + k + 1, V, dtype, 100 * B + k, masked)
    cfg = dict(B=B, k=k, max_new=max_new, greedy=greedy, seed=B)
    cfg.update(dict(svip=dict(h=1.3), constant=dict(h=math.inf), heuristic=dict(h=math.inf, gamma0=2, inc=2, dec=1))[policy])
    ref = _loop(svip, draft, target, one_by_one=True, **cfg)
    for chunk in (None, 1, 3):
        got = _loop(svip, draft, target, chunk=chunk, **cfg)
        for key in ("state", "out", "log"):
            assert torch.equal(ref[key], got[key]), (key, chunk)


def test_paused_loop_reports_as_before(svip):
    """Rounds in pieces: each call runs no more rounds than asked and says how many sequences are left."""
    draft, target = _trace(6, 40, 4000, torch.bfloat16, 7, False)
    a = svip.Loop(target, draft, temperature=1.0, h=1.3, gamma0=7, gamma_max=7, max_new=20, rounds=20, greedy=True)
    assert a.run(0) == (0, 6)
    seen = []
    while True:
        ran, running = a.run(2)
        seen.append((ran, running))
        assert running == int((a.state[:, 2] == 0).sum())
        if not running:
            break
        assert ran == 2
    assert a.run(3) == (0, 0)                                   # nothing is left to do
    done = a.state[:, 3].max().item()
    assert sum(r for r, _ in seen) == done and (a.round_log[done:] == -2).all()


@pytest.mark.parametrize("greedy", [True, False])
def test_workspace_for_single_positions(svip, greedy):
    """A workspace that holds a round's buffers but none for groups: position by position, with the same results, and nothing
    written behind it; one byte less is refused."""
    B, k, V, max_new = 5, 6, 9000, 12
    draft, target = _trace(B, max_new + k + 1, V, torch.float16, 11, False)
    up = lambda n: (n + 255) // 256 * 256
    least = up(svip.workspace_bytes(B, k, V)) + up(4 * B * k) + up(8 * B * k) + 2 * up(B) + 6 * up(4 * B) + 256
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    u = {} if greedy else dict(u_sample=torch.rand(max_new, B, k, device="cuda", generator=g),
                               u_accept=torch.rand(max_new, B, k, device="cuda", generator=g),
                               u_resample=torch.rand(max_new, B, device="cuda", generator=g))
    a, b = (svip.Loop(target, draft, temperature=1.0, h=1.3, gamma0=k, gamma_max=k, max_new=max_new, rounds=max_new,
                      greedy=greedy, **u) for _ in range(2))
    assert b.workspace.numel() > least
    b.workspace[least:] = 0xA5
    b.config.workspace_bytes = least - 1
    with pytest.raises(svip.SvipError):
        b.run()
    b.config.workspace_bytes = least
    ran, running = a.run()
    assert b.run() == (ran, running)
    assert torch.equal(a.state, b.state) and torch.equal(a.out_tokens, b.out_tokens)
    assert torch.equal(a.round_log[:ran], b.round_log[:ran])       # a round launched ahead may have filled its entries behind
    assert (b.workspace[least:] == 0xA5).all()
