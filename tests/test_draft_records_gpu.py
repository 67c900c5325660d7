"""The draft step at the sizes where its records change form: one and two records per lane of the finish, more tiles
than that, launches past the size up to which records keep their chunks' masses, rows that end inside a vector, a
chunk or a tile, masked tiles and extreme logits -- against the same quantities in fp64."""
import pytest
import torch

from helpers import MARGIN, REL

pytestmark = pytest.mark.gpu

BF, F16, F32 = torch.bfloat16, torch.float16, torch.float32
CASES = [
    (BF, 1, 1), (BF, 3, 8), (F16, 2, 513), (F32, 2, 1024), (BF, 2, 2047), (BF, 2, 2049),
    (BF, 2, 64 * 2048), (BF, 2, 64 * 2048 + 1), (F32, 2, 65 * 1024 - 3), (F16, 1, 75 * 2048 - 1664),     # two records per lane
    (BF, 1, 128 * 2048), (F32, 2, 128 * 1024 + 1), (BF, 1, 200 * 2048 + 9),                              # and more tiles than that
    (BF, 4100, 2048 + 520), (F32, 2701, 2 * 1024 + 7), (BF, 8101, 100), (F16, 8100, 100),               # around 8100 waves
]


def _rows(dtype, B, V, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    per16 = 4 if dtype == F32 else 8
    x = torch.empty(B, (V + per16 - 1) // per16 * per16, dtype=dtype, device="cuda")[:, :V]
    x.copy_(torch.randn(B, V, device="cuda", generator=g) * (1 + 4 * torch.rand(B, 1, device="cuda", generator=g)))
    return x, torch.rand(B, device="cuda", generator=g)


def _mask(p, *shape, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.rand(*shape, device="cuda", generator=g) < p


def _step(svip, x, u, T, greedy):
    B, V = x.shape
    o = dict(tok=torch.full((B,), -7, dtype=torch.int32, device="cuda"), ent=torch.empty(B, device="cuda"),
             q=torch.empty(B, device="cuda"), lse=torch.empty(B, dtype=torch.float64, device="cuda"),
             stop=torch.empty(B, dtype=torch.uint8, device="cuda"))
    svip.draft_step(x, temperature=T, h=1.5, step_j=0, k_max=4, u_sample=None if greedy else u, greedy=greedy,
                    token_out=o["tok"], entropy_out=o["ent"], q_tok_out=o["q"], lse_out=o["lse"], stop_out=o["stop"],
                    workspace=svip.new_workspace(B, 4, V))
    torch.cuda.synchronize()
    return o


def _check(o, x, u, T, greedy, q_rel=REL):
    V = x.shape[1]
    for b0 in range(0, x.shape[0], 512):
        s = slice(b0, b0 + 512)
        z = x[s].double() / T
        top = z.amax(-1, keepdim=True)
        lse0 = torch.logsumexp(z - top, -1)
        lse = lse0 + top[:, 0]
        p = torch.exp(z - top - lse0[:, None])
        H = -(p * torch.log(p.clamp_min(1e-300))).sum(-1)
        tok = o["tok"][s].long()
        assert (tok >= 0).all() and (tok < V).all()
        # a logsumexp sums fp32 weights of relative error 2^-22 in fp64; entropies and probabilities to the stated bar
        assert ((o["lse"][s] - lse).abs() <= 2.0 ** -22 * lse.abs().clamp_min(1.0)).all()
        assert ((o["ent"][s] - H).abs() <= REL * H + 1e-9).all()
        q = p.gather(1, tok[:, None])[:, 0]
        assert ((o["q"][s] - q).abs() <= q_rel * q).all()
        if greedy:
            assert torch.equal(tok, x[s].float().cpu().argmax(-1).to(tok.device))      # CPU argmax: the first maximum
        else:
            C = torch.cumsum(p, -1)
            hi = C.gather(1, tok[:, None])[:, 0]
            d = u[s].double() * C[:, -1]
            assert ((d < hi + 2 * MARGIN) & (d >= hi - q - 2 * MARGIN)).all() and (q > 0).all()
        sq = torch.sqrt(H)
        clear = (sq - 1.5).abs() >= MARGIN
        assert torch.equal(o["stop"][s][clear] != 0, (sq > 1.5)[clear])


@pytest.mark.parametrize("dtype,B,V", CASES)
def test_records_of_every_form(svip, dtype, B, V):
    x, u = _rows(dtype, B, V, seed=V + B)
    for greedy in (False, True):
        for T in (1.0, 0.7):
            _check(_step(svip, x, u, T, greedy), x, u, T, greedy)


@pytest.mark.parametrize("dtype", [BF, F16, F32])
@pytest.mark.parametrize("B,tiles", [(9, 5), (1400, 6)])
def test_masked_tiles_and_extreme_logits(svip, dtype, B, tiles):
    """Tiles that are masked but for one logit or altogether, rows of extremely negative logits, +0 beside -0 as
    the maximum, logits of extreme size; in one-tile and in two-tile records."""
    tile = 1024 if dtype == F32 else 2048
    V = tiles * tile - 11
    x, u = _rows(dtype, B, V, seed=5)
    low, big = (torch.finfo(dtype).min, 6e4) if dtype == F16 else (-1e38, 1e35)      # |z| log2(e) stays finite in fp32
    x[0, tile:3 * tile] = float("-inf")
    x[0, 2 * tile + 77] = 1.0
    x[2] = -3.0
    x[2, [tile + 4, 2 * tile + 9]] = 0.0
    x[2, tile + 2] = -0.0
    x[3] = float("-inf")
    x[3, V - 1] = 2.0
    if B < 100:                          # the workgroup search of two-tile records forms z c in fp32 before it subtracts
        x[1] = low
        x[1, tile:] = float("-inf")
        x[4, tile + 5] = big
        x[5] = -big
        x[5, 3] = -big * 0.5
    x[6:] = x[6:].where(x[6:] > 2.0, torch.full_like(x[6:], float("-inf")))
    x[6:, 17] = 3.0
    for greedy in (False, True):
        _check(_step(svip, x, u, 1.0, greedy), x, u, 1.0, greedy)


@pytest.mark.parametrize("dtype", [BF, F16, F32])
@pytest.mark.parametrize("B,tiles", [(9, 5), (1400, 6), (2, 64 * 34)])
def test_tiles_of_the_lowest_number(svip, dtype, B, tiles):
    """Masks of the type's most negative number, of -inf and of both (side by side in a vector, vector by vector, tile by
    tile), rows with few logits above them, in records of one, two and more tiles."""
    tile, low = 1024 if dtype == F32 else 2048, torch.finfo(dtype).min
    V = tiles * tile - 11
    x, u = _rows(dtype, B, V, seed=6)
    keep = _mask(0.3 / tile, B, V, seed=7)
    # one logit that none of the masks below takes away: a row of nothing but the lowest number has a token only where the
    # search subtracts before it multiplies, |low| log2(e) being more than fp32 holds
    keep[:, V // 32 * 16] = True
    x.copy_(x.where(keep, torch.full_like(x, low)))
    x[1, :V // 3] = float("-inf")
    if B > 2:
        x[2, 3::16] = float("-inf")
        x[3].view(-1)[: V // 16 * 16].view(-1, 16)[:, 8:] = float("-inf")
        x[4, :2 * tile] = low
        x[4, 2 * tile:] = 1.0
        x[5, :2 * tile] = 1.0
        x[5, 2 * tile:] = low
    if B < 100 and tiles < 100:          # the workgroup search of longer records forms z c in fp32 before it subtracts
        x[6] = low
        x[7] = float("-inf")
        x[7, tile + 8:3 * tile] = low
        x[8] = float("-inf")
        x[8, [tile + 9, 2 * tile + 3, V - 1]] = low
    for greedy in (False, True):
        _check(_step(svip, x, u, 1.0, greedy), x, u, 1.0, greedy)


@pytest.mark.parametrize("dtype", [BF, F16, F32])
@pytest.mark.parametrize("B,V", [(4, 50257), (4, 32768), (4100, 2048 + 520)])
def test_temperatures_near_zero(svip, dtype, B, V):
    """Accepted are all temperatures above 0.  Masked logits (-inf or the type's most negative number) and the places past
    the end of a ragged tile weigh nothing, whichever way log2(e) / T rounds to fp32: of these, some round up, some down."""
    for T in (1e-7, 1e-8, 1e-9, 1e-10, 3e-11, 1e-12):
        T = torch.tensor(T, dtype=torch.float32).item()          # the call takes the temperature in fp32
        x, u = _rows(dtype, B, V, seed=V + 3)
        x[1, _mask(0.3, V, seed=1)] = float("-inf")
        x[2, _mask(0.3, V, seed=2)] = torch.finfo(dtype).min
        # the workgroup search of launches beyond 8100 waves forms z c - L with L as two fp32 parts: two roundings of
        # at most |L| 2^-48 in the exponent of the token's weight
        q_rel = REL + (2.0 ** -47 * x.float().abs()[x > -1e4].max().item() / T if B > 4 else 0.0)
        for greedy in (False, True):
            _check(_step(svip, x, u, T, greedy), x, u, T, greedy, q_rel)


@pytest.mark.parametrize("B,V", [(6, 3 * 2048 + 77), (4100, 2048 + 520)])
@pytest.mark.parametrize("T", [1.0, 9.0, 12.0, 300.0, 3000.0])
def test_fp16_rows_near_the_lowest_number(svip, B, V, T):
    """fp16 has no room below -65504 in which a masked logit could stand for -inf next to logits around it."""
    x, u = _rows(F16, B, V, seed=V)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    low = (-65504.0 + 32.0 * torch.randint(0, 2, (2, V), device="cuda", generator=g)).half()
    x[0:2] = low.where(torch.rand(2, V, device="cuda", generator=g) < 0.01, torch.full_like(low, float("-inf")))
    x[1, :V // 2] = float("-inf")
    x[2, torch.rand(V, device="cuda", generator=g) < 0.5] = float("-inf")
    x[3, torch.rand(V, device="cuda", generator=g) < 0.5] = -65504.0
    # (see test_temperatures_near_zero for the second term)
    q_rel = REL + (2.0 ** -47 * 65504.0 / T if B > 6 else 0.0)
    for greedy in (False, True):
        _check(_step(svip, x, u, T, greedy), x, u, T, greedy, q_rel)


@pytest.mark.parametrize("dtype", [BF, F16, F32])
@pytest.mark.parametrize("B,tiles", [(4, 5), (1400, 6)])
def test_nan_logits_weigh_nothing(svip, dtype, B, tiles):
    """A NaN logit, of either sign, counts as a masked one: every output is that of the row with -inf in its place."""
    V = tiles * (1024 if dtype == F32 else 2048) - 11
    x, u = _rows(dtype, B, V, seed=8)
    at = _mask(0.001, 3, V, seed=3)
    at[2, :V // 2] = True
    x[:3] = x[:3].masked_fill(at, float("-inf"))
    word, quiet = {BF: (torch.int16, 0x7FC0), F16: (torch.int16, 0x7E00), F32: (torch.int32, 0x7FC00000)}[dtype]
    for nan in (quiet, quiet + torch.iinfo(word).min):
        y, _ = _rows(dtype, B, V, seed=8)
        y.copy_(x)
        bits = y.view(word)
        bits[:3] = bits[:3].masked_fill(at, nan)
        assert torch.isnan(y[:3][at]).all()
        for greedy in (False, True):
            _check(_step(svip, y, u, 1.0, greedy), x, u, 1.0, greedy)


@pytest.mark.parametrize("dtype", [BF, F16, F32])
@pytest.mark.parametrize("B,V", [(4, 5 * 2048 - 11), (4, 70 * 2048), (1400, 6 * 2048)])
def test_rows_without_a_distribution_have_no_token(svip, dtype, B, V):
    """Rows with a logit of +inf, in the first or in a later record, and rows without a finite one: token -1."""
    x, u = _rows(dtype, B, V, seed=9)
    u[:] = torch.linspace(0, 0.999, B, device="cuda")
    x[0, 3] = float("inf")
    x[1, V - 5] = float("inf")
    x[2, [5, V // 2]] = float("inf")
    x[3] = float("-inf")
    o = _step(svip, x, u, 1.0, False)
    assert (o["tok"][:4] == -1).all() and torch.isnan(o["q"][:4]).all() and (o["stop"][:4] == 0).all()
    _check({n: t[4:] for n, t in o.items()}, x[4:], u[4:], 1.0, False)


@pytest.mark.parametrize("B,V,greedy", [(64, 6 * 2048 - 40, False), (64, 70 * 2048, False), (64, 6 * 2048, True), (1400, 6 * 2048, False)])
def test_stop_flags_in_place_and_apart(svip, B, V, greedy):
    """A step that reads and writes one array of flags gives, bit for bit, what it gives with two arrays, where rows are
    already stopped, stop by their entropy, and all stop at the cap."""
    x, u = _rows(BF, B, V, seed=10)
    ws = svip.new_workspace(B, 4, V)
    before = (torch.arange(B, device="cuda") % 5 == 3).to(torch.uint8)

    def step(flags_in, flags_out, j):
        o = dict(tok=torch.full((B,), -7, dtype=torch.int32, device="cuda"), ent=torch.zeros(B, device="cuda"),
                 q=torch.zeros(B, device="cuda"), lse=torch.zeros(B, dtype=torch.float64, device="cuda"),
                 len=torch.zeros(B, dtype=torch.int32, device="cuda"), stop=flags_out)
        svip.draft_step(x, temperature=1.0, h=1.4, step_j=j, k_max=4, u_sample=None if greedy else u, greedy=greedy,
                        stop_in=flags_in, token_out=o["tok"], entropy_out=o["ent"], q_tok_out=o["q"], lse_out=o["lse"],
                        stop_out=o["stop"], draft_len_out=o["len"], workspace=ws)
        torch.cuda.synchronize()
        return o

    for j in (1, 3):
        apart = step(before, torch.full_like(before, 9), j)
        live = before == 0
        assert (apart["tok"][live] >= 0).all() and (apart["tok"][~live] == -1).all() and (apart["stop"][~live] == 1).all()
        assert (apart["stop"][live] == 1).all() if j == 3 else 0 < apart["stop"][live].sum() < live.sum()
        for _ in range(20):
            flags = before.clone()
            same = step(flags, flags, j)
            assert all(torch.equal(same[n], apart[n]) for n in apart)


# Steps of one launch against two launches over the same records (a forced count takes those): rows of one to 64 records, whole
# and partial workgroups and rounds of the XCDs, just inside and outside the line between the forms.
ONE_LAUNCH = [(BF, 1, 100), (F32, 9, 1024 + 1), (F16, 7, 3 * 2048), (BF, 8, 4 * 2048 + 8), (F32, 17, 5 * 1024 - 1), (BF, 3, 63 * 2048 + 77),
              (F32, 2, 64 * 1024), (BF, 190, 13 * 2048 + 5), (BF, 260, 13 * 2048 + 5), (F32, 96, 31 * 1024 + 9), (BF, 768, 700), (BF, 1030, 700)]


@pytest.mark.parametrize("dtype,B,V", ONE_LAUNCH)
def test_one_launch_gives_what_two_give(svip, dtype, B, V):
    """Bit for bit, over a chain of three steps whose stop flags are updated in place (some rows stopped before it, others on the
    way), in a workspace that the same steps have used before."""
    records = -(-V // (1024 if dtype == F32 else 2048))
    rows = [_rows(dtype, B, V, seed=31 * V + j) for j in range(3)]
    ws = svip.new_workspace(B, 3, V)
    got = []
    try:
        for forced in (0, 0, records):
            svip.bench_set_tuning(draft_slices=forced)
            for greedy in (False, True):
                o = {n: torch.full((B, 3), -7, dtype=t, device="cuda") for n, t in
                     (("tok", torch.int32), ("ent", F32), ("q", F32), ("lse", torch.float64))}
                stop, dlen = torch.zeros(B, dtype=torch.uint8, device="cuda"), torch.full((B,), -7, dtype=torch.int32, device="cuda")
                stop[1::5] = 1
                for j, (x, u) in enumerate(rows):
                    svip.draft_step(x, temperature=0.9, h=1.3, step_j=j, k_max=4, greedy=greedy,
                                    u_sample=None if greedy else u[:, None].expand(B, 3).contiguous()[:, j], stop_in=stop,
                                    token_out=o["tok"][:, j], entropy_out=o["ent"][:, j], q_tok_out=o["q"][:, j],
                                    lse_out=o["lse"][:, j], stop_out=stop, draft_len_out=dlen, workspace=ws)
                torch.cuda.synchronize()
                got.append(dict(o, stop=stop, dlen=dlen))
    finally:
        svip.bench_set_tuning()
    for i in range(4):
        for n, want in got[4 + i % 2].items():
            assert torch.equal(got[i][n], want), (i, n)


@pytest.mark.parametrize("dtype,B,V", [(BF, 5, 65 * 2048 - 9), (F16, 19, 70 * 2048), (BF, 2, 128 * 2048), (F32, 8, 100 * 1024 + 3)])
def test_one_launch_two_records_per_lane(svip, dtype, B, V):
    x, u = _rows(dtype, B, V, seed=V + B)
    for greedy in (False, True):
        _check(_step(svip, x, u, 0.8, greedy), x, u, 0.8, greedy)
