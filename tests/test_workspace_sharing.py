"""Calls of different sizes in one workspace.  Its last part holds counters that calls hand rows over with, and each call's own data grows
from the front: what a call lays over the counters of a larger batch than its own."""
import bisect
import itertools
import math
import random

import pytest
import torch

import paper_2411_18462_amd as svip

F32, BF = torch.float32, torch.bfloat16
VEC = {F32: 4, BF: 8}
DRAFT, VERIFY, VERIFY_RE, GREEDY, PAIR, PAIR_RE = range(6)


def _up(n):
    return (n + 255) // 256 * 256


def _counters(rows):
    return _up(64 * rows)


def _front(call, dtype, B, k, V):
    """Where a call's data ends: what it needs less its counters.  Slice statistics are counted with 24 bytes and have 16; the slices here
    are those of the diagnostics (svip_kernels.hip, make_geo), checked against the size itself."""
    need = svip.workspace_needed(call, dtype, B, k, V) - _counters(B)
    if call not in (PAIR, PAIR_RE):
        return need

    def slices(rows):
        tiles = -(-V // (256 * VEC[dtype]))
        ns = max(1, min(-(-8192 // rows), tiles // 8, 64))
        per = -(-tiles // ns)
        return -(-tiles // (per + (per > 1 and per % 2 == 0)))

    rows, pos = B * (k + 1 + (k if call == PAIR_RE else 0)), B * k
    stats, rest = rows * slices(rows), 256 + _up(24 * B) + _up(16 * pos) + _up(24 * pos * slices(pos))
    assert need == rest + _up(24 * stats)
    return rest + _up(16 * stats)


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def test_workspaces_of_the_largest_sizes_keep_every_counter():
    rng = random.Random(1)
    for _ in range(20000):
        most = _log(rng, 1, 4096), _log(rng, 1, 1024), _log(rng, 1, 400000)
        B, k, V = (_log(rng, 1, m) for m in most)
        call, dtype = rng.randrange(6), rng.choice([F32, BF])
        if svip.workspace_needed(call, dtype, B, k, V):
            assert _front(call, dtype, B, k, V) <= svip.workspace_bytes(*most) - _counters(most[0]), (call, dtype, B, k, V, most)


def test_draft_counters_where_every_call_has_its_workspace_bytes():
    """A draft step of at most 1024 workgroups uses its rows' counters where the workspace has svip_workspace_bytes of its sizes: no call
    that has as much reaches them, whatever its batch, drafts and vocabulary are."""
    rng = random.Random(2)
    steps = sorted((svip.workspace_bytes(B, k, V), B) for B, k, V in
                   ((_log(rng, 1, 1024), rng.choice([1, 1, _log(rng, 1, 64)]), _log(rng, 1, 160000)) for _ in range(4000)))
    sizes, rows_of = [size for size, _ in steps], list(itertools.accumulate((B for _, B in steps), max))
    looked = 0
    for _ in range(60000):
        B, k, V = _log(rng, 1, 1024), _log(rng, 1, 1024), _log(rng, 1, 400000)
        call, dtype = rng.randrange(6), rng.choice([F32, BF])
        mine = svip.workspace_bytes(B, k, V)
        fits = bisect.bisect_right(sizes, mine)
        rows = rows_of[fits - 1] if fits else 0
        if rows > B and svip.workspace_needed(call, dtype, B, k, V):
            looked += 1
            assert _front(call, dtype, B, k, V) <= mine - _counters(rows), (call, dtype, B, k, V, rows)
    assert looked > 10000


STEPS = [                                    # sharing a workspace of what the larger of the two needs
    (F32, (7, 2000), (4, 8000)),             # one workgroup per row
    (F32, (5, 5000), (1, 32000)),            # two
    (BF, (24, 20000), (3, 128256)),          # three and sixteen
    (BF, (64, 32000), (20, 100000)),
]


@pytest.mark.gpu
@pytest.mark.parametrize("greedy", [False, True])
@pytest.mark.parametrize("dtype,a,b", STEPS)
def test_draft_steps_of_two_sizes_in_the_larger_one_s_workspace(svip, dtype, a, b, greedy):
    """As in workspaces of their own, in any order and with anything in the workspace behind its flag word."""
    print(f"sharing {dtype} {a} {b} greedy={greedy}", flush=True)
    k, g = 4, torch.Generator(device="cuda").manual_seed(a[0])
    size = max(svip.workspace_needed(DRAFT, dtype, B, k, V) for B, V in (a, b))
    shared = torch.empty(size, dtype=torch.uint8, device="cuda")
    svip.load().svip_workspace_reset(shared.data_ptr(), size, None)
    calls = []
    for B, V in (a, b):
        x = torch.empty(B, -(-V // 8) * 8, dtype=dtype, device="cuda")[:, :V]
        x.copy_(torch.randn(B, V, device="cuda", generator=g) * 4)
        calls.append((x, torch.rand(B, device="cuda", generator=g)))

    def step(x, u, ws):
        B, V = x.shape
        o = dict(token_out=torch.full((B,), -9, dtype=torch.int32, device="cuda"), entropy_out=torch.full((B,), -9.0, device="cuda"),
                 q_tok_out=torch.full((B,), -9.0, device="cuda"), lse_out=torch.full((B,), -9.0, dtype=torch.float64, device="cuda"),
                 stop_out=torch.full((B,), 9, dtype=torch.uint8, device="cuda"), draft_len_out=torch.full((B,), -9, dtype=torch.int32, device="cuda"))
        svip.draft_step(x, temperature=1.0, h=1.5, step_j=1, k_max=k, greedy=greedy, u_sample=None if greedy else u, workspace=ws, **o)
        torch.cuda.synchronize()
        return o

    want = [step(x, u, svip.new_workspace(x.shape[0], k, x.shape[1])) for x, u in calls]
    for i in (0, 1, 0, 0, 1):
        got = step(*calls[i], shared)
        for n in want[i]:
            assert torch.equal(got[n], want[i][n]), (i, n)
        if i:
            shared[256:] = 0xA5
