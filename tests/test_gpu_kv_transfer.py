"""GPU: cache export and import move 8 elements at a time when the caller's arrays allow it and one at a time when they do
not: both must be bit-exact for every kind of cache, head size and remainder of a 64-token block."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _offset(t, by):
    """The same values in a contiguous tensor that starts `by` elements into its storage."""
    buf = torch.empty(t.numel() + by, dtype=t.dtype, device=t.device)
    v = buf[by:].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("n", [1, 7, 63, 64, 65, 200])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", ["contiguous", "paged", "fp8", "paged_fp8"])
@pytest.mark.parametrize("by", [0, 1])
def test_round_trips_are_exact(kind, d, n, by):
    from paper_2509_24381_amd import runner
    from paper_2509_24381_amd.binding import _check, _ptr, KVPool
    shape = synth.LayerShape("kv", 256, 6, 3, d, 256)
    ctx = runner.Context(runner.config_for(shape, max_tokens=64, max_requests=1, max_pos=512))
    g = torch.Generator(device="cuda").manual_seed(n + d)
    rows = [torch.randn((n, 3, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2)]
    if kind.startswith("paged"):
        kv = KVPool(ctx, 6, fp8=kind == "paged_fp8").new_cache(1, 0.125, 0.25)
    else:
        kv = ctx.kv_alloc_fp8(1, 256, 0.125, 0.25) if kind == "fp8" else ctx.kv_alloc(1, 256)
    kv.slab.fill_(0xFF)                       # NaN patterns: what import must clear shows up in the V^T tail
    kv.import_(0, *(_offset(t, by) for t in rows))
    stream = torch.cuda.current_stream().cuda_stream or None
    out = [_offset(torch.zeros_like(t), by) for t in rows]
    _check(ctx.lib.rs_kv_export(kv.handle, 0, _ptr(out[0]), _ptr(out[1]), stream))
    want = rows
    if "fp8" in kind:
        want = [((r.float() / s).clamp(-448, 448).to(torch.float8_e4m3fn).float() * s).to(torch.bfloat16)
                for r, s in zip(rows, (0.125, 0.25))]           # (the scales are powers of two: the division is exact)
        codes = [_offset(torch.zeros(t.shape, dtype=torch.uint8, device="cuda"), by) for t in rows]
        _check(ctx.lib.rs_kv_export_codes(kv.handle, 0, _ptr(codes[0]), _ptr(codes[1]), stream))
        for c, r, s in zip(codes, rows, (0.125, 0.25)):
            assert torch.equal(c, (r.float() / s).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8))
        kv.slab.fill_(0xFF)
        kv.reset()
        kv.import_codes(0, codes[0], codes[1])
        again = [torch.zeros_like(t) for t in rows]
        _check(ctx.lib.rs_kv_export(kv.handle, 0, _ptr(again[0]), _ptr(again[1]), stream))
        assert all(torch.equal(a.view(torch.int16), w.view(torch.int16)) for a, w in zip(again, want))
    assert all(torch.equal(o.view(torch.int16), w.view(torch.int16)) for o, w in zip(out, want))
    tail = -n % 64
    if tail and kind == "contiguous":         # V^T places behind the last token read as zeros
        v = kv.slab.view(torch.int16)[3 * 256 * d: 2 * 3 * 256 * d].view(3, 4, d, 64)
        assert bool((v[:, (n - 1) // 64, :, 64 - tail:] == 0).all())
    del kv
