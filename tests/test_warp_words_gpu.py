"""The filter's comparison of stored words (thresholds that are zero of either sign, next to the ends of a type, or keep
everything) and its way past the caches for calls larger than they are."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

BITS = {torch.float32: torch.int32, torch.bfloat16: torch.int16, torch.float16: torch.int16}


def _rows(x):
    """A copy of x [rows, V] as a [1, rows, V] view whose rows start on 16-byte boundaries."""
    per16 = 16 // x.element_size()
    V = x.shape[1]
    buf = torch.zeros(1, x.shape[0], (V + per16 - 1) // per16 * per16, dtype=x.dtype, device="cuda")
    buf[0, :, :V] = x
    return buf[:, :, :V]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("V", [1, 7, 8, 1023, 8195, 40001])
@pytest.mark.parametrize("shortcut", [True, False])
def test_thresholds_at_special_values(svip, dtype, V, shortcut):
    print(f"warp words {dtype} V={V} shortcut={shortcut}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(V)
    low, high, tiny = torch.finfo(dtype).min, torch.finfo(dtype).max, torch.finfo(dtype).smallest_normal
    values = torch.tensor([-math.inf, low, -1.0, -tiny, -0.0, 0.0, tiny, 1.0, high], device="cuda")
    picks = values[torch.randint(0, len(values), (12, V), device="cuda", generator=g)]
    picks[0] = -0.0
    picks[1] = 0.0
    picks[2] = low
    picks[3] = -math.inf
    picks[3, V // 2] = 0.5
    x = picks.to(dtype)
    src = _rows(x)
    try:
        svip.bench_set_tuning(warp_no_shortcut=0 if shortcut else 1)
        for k in sorted({1, 2, max(1, V // 5), max(1, V // 2), V - 1, V}):
            if k < 1:
                continue
            out, kept = _rows(torch.zeros_like(x)), torch.zeros(12, dtype=torch.int32, device="cuda")
            svip.warp_logits(src, temperature=1.0, top_k=k, out=out, kept_out=kept)
            inplace = _rows(x)
            svip.warp_logits(inplace, temperature=1.0, top_k=k)
            torch.cuda.synchronize()
            keep = torch.ones_like(x, dtype=torch.bool) if k >= V else x.float() >= x.float().topk(k, dim=1).values[:, -1:]
            want = torch.where(keep, x, torch.full_like(x, -math.inf))
            assert torch.equal(out[0].contiguous().view(BITS[dtype]), want.view(BITS[dtype])), k       # signs of zeros too
            assert torch.equal(inplace[0].contiguous().view(BITS[dtype]), want.view(BITS[dtype])), k
            assert torch.equal(kept.long(), keep.sum(1)), k
    finally:
        svip.bench_set_tuning()


@pytest.mark.parametrize("dtype,V,top_k,top_p", [(torch.bfloat16, 131075, 0, 0.9), (torch.float32, 98308, 0, 0.9), (torch.float16, 131080, 50, 0.9),
                                                (torch.float32, 70001, 600, 1.0), (torch.bfloat16, 131075, 0, 1.0)])
def test_calls_larger_than_the_caches_equal_smaller_ones(svip, dtype, V, top_k, top_p):
    rows = int(150e6 / (V * (4 if dtype == torch.float32 else 2)))
    print(f"warp past the caches {dtype} V={V} rows={rows} top_k={top_k} top_p={top_p}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(V)
    x = torch.empty(rows, V, dtype=dtype, device="cuda")
    for r in range(0, rows, 64):
        n = min(64, rows - r)
        x[r:r + n] = torch.randn(n, V, device="cuda", generator=g) * (1.0 + 5.0 * torch.rand(n, 1, device="cuda", generator=g))
    src = _rows(x)
    out, kept = _rows(torch.zeros_like(x)), torch.zeros(rows, dtype=torch.int32, device="cuda")
    svip.warp_logits(src, temperature=1.0, top_k=top_k, top_p=top_p, out=out, kept_out=kept)
    for r in range(0, rows, 128):
        part, few = _rows(x[r:r + 128]), torch.zeros(min(128, rows - r), dtype=torch.int32, device="cuda")
        ref = _rows(torch.zeros_like(x[r:r + 128]))
        svip.warp_logits(part, temperature=1.0, top_k=top_k, top_p=top_p, out=ref, kept_out=few)
        torch.cuda.synchronize()
        assert torch.equal(ref.contiguous().view(BITS[dtype]), out[:, r:r + 128].contiguous().view(BITS[dtype])), r
        assert torch.equal(few, kept[r:r + 128]), r
