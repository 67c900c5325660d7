"""The decoding loop with several draft positions per launch against the loop that takes them one by one (which it still does
in large batches, and where an override asks for records of another size): state, tokens and log are the
same bit for bit.  64 records per row, the override used here, is what the rows of these shapes have anyway, so both sides
sum the same partial results."""
import math
from types import SimpleNamespace

import pytest
import torch

from test_loop_gpu import _check

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


def _rows_with_ties(B, L, V, dtype, seed):
    """Traces whose maxima lie in every part of a row: ties in the first, a middle and the last tile, in two of the last tiles, a
    single one in the row's last logit; heavy-tailed rows in between."""
    draft, target = _trace(B, L, V, dtype, seed, False)
    tile = 256 * (16 // draft.element_size())
    for t, at in ((draft, 0), (target, 1)):
        top = t.amax(-1, keepdim=True)
        for j0, cols in ((1, [5, V // 2, V - 1]), (2, [V - 1 - 2 * tile, V - 1 - tile, V - 1]), (3, [V - 1])):
            rows = slice((j0 + at) % 5, None, 5)
            t[:, rows, cols] = top[:, rows] + (0.5 if dtype != torch.float16 else 1.0)
    return draft, target


@pytest.mark.parametrize("greedy", [True, False])
@pytest.mark.parametrize("B,V,dtype", [
    (9, 151936, torch.bfloat16),         # 75 tiles: two records per lane of the finish
    (2, 65537, torch.float32),           # 65 tiles, the last with one logit: the second record of lane 32 is the last
    (3, 151936, torch.float32),          # 149 tiles: three records per lane
    (1, 262145, torch.float16),          # 129 tiles, one logit in the last
    (2, 196608, torch.float32),          # 192 tiles, the most that are taken in groups
])
def test_rows_of_several_records_per_lane(svip, B, V, dtype, greedy):
    """Round by round against the oracle; up to 128 tiles also bit for bit against the loop that takes positions one by one (beyond,
    svip_draft_step keeps one sum for several tiles, and the two agree to rounding)."""
    print(f"loop records B={B} V={V} {dtype} greedy={greedy}", flush=True)
    k, max_new = 6, 10
    draft, target = _rows_with_ties(B, max_new + k + 1, V, dtype, V + B)
    g = torch.Generator(device="cuda").manual_seed(B)
    u = dict(u_sample=torch.rand(max_new, B, k, device="cuda", generator=g), u_accept=torch.rand(max_new, B, k, device="cuda", generator=g),
             u_resample=torch.rand(max_new, B, device="cuda", generator=g))
    h = 1.5
    results = []
    for small in (False, True):
        loop = svip.Loop(target, draft, temperature=1.0, h=h, gamma0=k, gamma_max=k, max_new=max_new, rounds=max_new, greedy=greedy,
                         **({} if greedy else u))
        if small:
            up = lambda n: (n + 255) // 256 * 256
            loop.config.workspace_bytes = up(svip.workspace_bytes(B, k, V)) + up(4 * B * k) + up(8 * B * k) + 2 * up(B) + 6 * up(4 * B) + 256
        ran, running = loop.run()
        assert running == 0 and loop.flags() == 0 and ran == int(loop.state[:, 3].max())
        results.append(dict(state=loop.state.cpu().numpy(), out=loop.out_tokens.cpu().numpy(), log=loop.round_log.cpu().numpy()[:ran], rounds=ran))
    tiles = -(-V // (256 * (16 // draft.element_size())))
    if tiles <= 128:
        assert results[0]["rounds"] == results[1]["rounds"]
        for key in ("state", "out", "log"):
            assert (results[0][key] == results[1][key]).all(), key
    rows = slice(0, 3)
    trace = dict(draft=draft[rows].float().cpu(), target=target[rows].float().cpu(), u_sample=u["u_sample"][:, rows].cpu(),
                 u_accept=u["u_accept"][:, rows].cpu(), u_resample=u["u_resample"][:, rows].cpu())
    for res in results:
        part = dict(state=res["state"][rows], out=res["out"][rows], log=res["log"][:, rows], rounds=res["rounds"])
        st = _check(part, trace, SimpleNamespace(T=1.0), (h, k, k, 0, 0), max_new, greedy=greedy)
        print("  ", st, flush=True)
        assert st["rounds"] >= 2 * min(B, 3) and (not greedy or st["free_checked"] == min(B, 3))


def _least_workspace(svip, B, k, V):
    """The least that rows are read ahead with (plan_groups and plan_bytes in svip_loop.hip): the records of the sampling loop's largest
    group, which a greedy launch shares its rows and keys into, and the same of a small greedy launch."""
    up = lambda n: (n + 255) // 256 * 256
    lanes, most = B if B < 8 else (B + 7) // 8 * 8, 0
    for vec in (4, 8):
        tiles = -(-V // (256 * vec))
        first, small = (min(k, max(2, n // (B * tiles))) for n in (4800, min(2400, 64 * B * tiles)))
        largest = max(first, min(k, 32768 // (tiles * ((B + 7) // 8 * 8))))
        most = max(most, up(lanes * largest * tiles * 64), up(lanes * small * tiles * 32) + up(lanes * (small + 1) * tiles * 8))
    serial = up(svip.workspace_bytes(B, k, V)) + up(4 * B * k) + up(8 * B * k) + 2 * up(B) + 6 * up(4 * B) + 256
    return serial + 2 * up(4 * B) + up(4 * B * (k + 1)) + most


@pytest.mark.parametrize("B,k,V,L,max_new,h,policy,workspace", [
    (2, 200, 600, 420, 210, math.inf, (200, 0, 0), "full"),      # drafts longer than a launch's rows; all but a few rows accepted
    (3, 300, 72, 700, 390, 4.0, (300, 0, 0), "full"),            # stops here and there, drafts of up to 300
    (64, 30, 65536, 64, 40, math.inf, (3, 7, 2), "least"),       # growing limits, drafts of several launches of 12 rows
    (5, 64, 400, 150, 200, math.inf, (64, 0, 0), "full"),        # the trace ends before max_new
    (9, 1, 2500, 40, 38, 1.0, (1, 0, 0), "least"),               # drafts of one token, one row per launch
    (4, 20, 300, 60, 30, 9.0, (20, 0, 0), "unfinished"),         # rows without any maximum: tokens of -1 are flagged and accepted
])
def test_greedy_rows_read_ahead(svip, B, k, V, L, max_new, h, policy, workspace):
    """The greedy loop reads rows far ahead of its rounds: the same as position by position wherever launches end, for a whole run
    and for one in pieces."""
    print(f"loop ahead B={B} k={k} V={V} L={L} {policy} {workspace}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(V)
    draft = (torch.randn(B, L, V, device="cuda", generator=g) * (1.0 + 5.0 * torch.rand(B, L, 1, device="cuda", generator=g)))
    target = draft.clone()
    other = torch.rand(B, L, device="cuda", generator=g) < 0.03
    target[other] = target[other].roll(1, -1)                              # another argmax in these rows
    if workspace == "unfinished":
        draft[:, 7::9] = target[:, 7::9] = -math.inf
    results = []
    for one_by_one, chunk in ((True, None), (False, None), (False, 1), (False, 5)):
        try:
            if one_by_one:
                svip.bench_set_tuning(draft_slices=64)
            loop = svip.Loop(target, draft, temperature=1.0, h=h, gamma0=policy[0], gamma_max=k, gamma_inc=policy[1], gamma_dec=policy[2],
                             max_new=max_new, rounds=max_new, greedy=True)
            if workspace == "least" and not one_by_one:
                loop.config.workspace_bytes = _least_workspace(svip, B, k, V)
                assert loop.config.workspace_bytes < loop.workspace.numel()
            ran, running = 0, 1
            while running and loop.next_round < max_new:
                n, running = loop.run(chunk)
                ran += n
        finally:
            svip.bench_set_tuning()
        assert running == 0 and ran == int(loop.state[:, 3].max())
        results.append((loop.state.cpu(), loop.out_tokens.cpu(), loop.round_log.cpu()[:ran], loop.flags()))
    assert (results[0][3] != 0) == (workspace == "unfinished")
    if workspace == "least":
        _launches_of_the_least_workspace(svip, draft, target, B, k, V, max_new, h, policy)
    for got in results[1:]:
        for x, y in zip(results[0][:3], got[:3]):
            assert torch.equal(x, y)
        assert got[3] == results[0][3]


def _launches_of_the_least_workspace(svip, draft, target, B, k, V, max_new, h, policy):
    """Pairs of launches of a whole run: with the least workspace more than with all of it, and with a byte less the loop goes position
    by position."""
    least, used = _least_workspace(svip, B, k, V), []
    for size in (None, least, least - 256):
        loop = svip.Loop(target, draft, temperature=1.0, h=h, gamma0=policy[0], gamma_max=k, gamma_inc=policy[1], gamma_dec=policy[2],
                         max_new=max_new, rounds=max_new, greedy=True)
        loop.config.workspace_bytes = size or loop.config.workspace_bytes
        events = [[torch.cuda.Event(enable_timing=True) for _ in range(2000)] for _ in range(2)]
        for e in events[0] + events[1]:
            e.record()                            # creates it
        keep = svip.bench_time_kernels(0, *[[e.cuda_event for e in es] for es in events])      # k_stream_rows; else the steps' statistics
        try:
            loop.run()
            used.append(svip.bench_events_used(0))
        finally:
            svip.bench_time_kernels(0, [], [])
        del keep
    rounds = int(loop.state[:, 3].max())
    print("  launches", used, "rounds", rounds, flush=True)
    assert used[0] < used[1] <= used[2] and used[2] >= rounds
    if k > 1:
        assert used[1] < used[2] and used[1] >= -(-max_new // 12)


@pytest.mark.parametrize("later", [0, 3, 17])
def test_a_later_call_asks_for_fewer_tokens(svip, later):
    """Sequences that have all the tokens a call asks for, but were not finished by the calls before it, go through one more round."""
    B, k, V, max_new, L = 5, 6, 700, 40, 60
    draft, target = _trace(B, L, V, torch.bfloat16, 21, False)
    results = []
    for one_by_one in (True, False):
        try:
            if one_by_one:
                svip.bench_set_tuning(draft_slices=64)
            loop = svip.Loop(target, draft, temperature=1.0, h=1.5, gamma0=k, gamma_max=k, max_new=max_new, rounds=max_new, greedy=True)
            ran = [loop.run(8)]
            before = loop.state.clone()
            loop.config.max_new = later
            ran += [loop.run(1), loop.run()]
        finally:
            svip.bench_set_tuning()
        assert ran[0][0] == 8 and ran[2][1] == 0 and (before[:, 6] > later + (0 if later == 17 else k)).any() and (before[:, 2] == 0).all()
        results.append((ran, loop.state.cpu(), loop.out_tokens.cpu(), loop.round_log.cpu()[:int(loop.state[:, 3].max())]))
    assert results[0][0] == results[1][0]
    for x, y in zip(results[0][1:], results[1][1:]):
        assert torch.equal(x, y)


@pytest.mark.parametrize("greedy", [True, False])
def test_limits_set_between_calls(svip, greedy):
    """A caller with a rule of its own stores the next round's limits into the state; one above gamma_max drafts gamma_max positions, is
    logged as it stands and counted down from."""
    B, k, V, max_new = 6, 5, 900, 24
    draft, target = _trace(B, 60, V, torch.float16, 33, False)
    g = torch.Generator(device="cuda").manual_seed(4)
    u = {} if greedy else dict(u_sample=torch.rand(max_new, B, k, device="cuda", generator=g),
                               u_accept=torch.rand(max_new, B, k, device="cuda", generator=g),
                               u_resample=torch.rand(max_new, B, device="cuda", generator=g))
    limits = torch.tensor([[1, 2, 3, 5, 7, 9], [9, 6, 4, 3, 2, 1]], dtype=torch.int32, device="cuda")
    results = []
    for one_by_one in (True, False):
        try:
            if one_by_one:
                svip.bench_set_tuning(draft_slices=64)
            loop = svip.Loop(target, draft, temperature=1.0, h=math.inf, gamma0=k, gamma_max=k, gamma_inc=2, gamma_dec=1, max_new=max_new,
                             rounds=max_new, greedy=greedy, **u)
            for n in (1, 2):
                loop.run(n)
                loop.state[:, 1] = limits[n - 1]
            loop.run()
        finally:
            svip.bench_set_tuning()
        rounds = int(loop.state[:, 3].max())
        assert (loop.state[:, 2] == 1).all() and (loop.round_log[:rounds, :, 1] > k).any()
        results.append((loop.state.cpu(), loop.out_tokens.cpu(), loop.round_log.cpu()[:rounds]))
    for x, y in zip(*results):
        assert torch.equal(x, y)
