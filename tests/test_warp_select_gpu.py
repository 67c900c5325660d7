"""The filter's threshold among a list's candidates, by digits as fine as their span allows, and the sweep that lists them by the sign of
the pivot: bit for bit what the histograms over the whole row give, for rows on either side of zero and of every span."""
import pytest
import torch

pytestmark = pytest.mark.gpu

BF, F16, F32 = torch.bfloat16, torch.float16, torch.float32
ROWS = ["positive", "negative", "around zero", "tiny", "wide", "two values", "few", "one"]


def _row(kind, V, g):
    z = torch.randn(V, device="cuda", generator=g) * 5
    if kind == "positive":
        return z + 60
    if kind == "negative":
        return z - 60
    if kind == "tiny":                       # subnormal in fp16
        return z * 1e-6
    if kind == "wide":                       # candidates of one sign and of many binades
        return z.sign() * torch.exp2(z.abs())
    if kind == "two values":
        return torch.where(z > 8, 1.0, -0.0)
    if kind == "few":
        return torch.where(z > 14, z, float("-inf"))
    if kind == "one":
        return torch.where(torch.arange(V, device="cuda") == V // 3, 3.0, -200.0)
    return z - 20                            # the pivot lies around zero


@pytest.mark.parametrize("dtype", [BF, F16, F32])
@pytest.mark.parametrize("V", [98304, 100003])
def test_thresholds_of_lists_equal_those_of_histograms(svip, dtype, V):
    g = torch.Generator(device="cuda").manual_seed(V)
    per16 = 4 if dtype == F32 else 8
    stride = -(-V // per16) * per16
    bits = torch.int32 if dtype == F32 else torch.int16

    def rows():
        return torch.empty(1, len(ROWS), stride, dtype=dtype, device="cuda")[:, :, :V]

    x = rows()
    for i, kind in enumerate(ROWS):
        x[0, i] = _row(kind, V, g).clamp(-6e4, 6e4) if kind != "few" else _row(kind, V, g)
    try:
        for T, k, p in ((1.0, 0, 0.9), (0.7, 0, 0.3), (2.0, 0, 0.5), (1.0, 50, 1.0), (1.0, 50, 0.9), (1.0, 1, 1.0), (0.8, 900, 0.95)):
            got = []
            for forced in (1, 0):
                svip.bench_set_tuning(warp_no_shortcut=forced)
                out, kept = rows(), torch.zeros(len(ROWS), dtype=torch.int32, device="cuda")
                svip.warp_logits(x, temperature=T, top_k=k, top_p=p, out=out, kept_out=kept)
                torch.cuda.synchronize()
                got.append((out.contiguous().view(bits), kept))
            for i, kind in enumerate(ROWS):
                assert torch.equal(got[0][0][0, i], got[1][0][0, i]), (kind, T, k, p)
            assert torch.equal(got[0][1], got[1][1]), (T, k, p)
    finally:
        svip.bench_set_tuning()
