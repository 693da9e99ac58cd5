"""GPU: projections whose weights are loaded with the streaming hint."""
import functools

import numpy as np
import pytest

import synth
from oracle import ChunkedPrefill, LayerParams
from test_gpu_parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_cu", [None, "200"])
def test_weights_that_are_streamed(n_cu, monkeypatch):
    """Matrices of 32 MB and more in calls of one block of rows, whose loads carry the streaming hint."""
    from paper_2509_24381_amd import runner as r
    if n_cu:
        monkeypatch.setenv("RS_NCU", n_cu)
    shape = synth.LayerShape("streamed", 2048, 4, 2, 128, 8448)
    w = synth.layer_weights(shape, 95, qkv_bias=True, gains="uniform")
    x = synth.prompt_rows([("image", 128)], shape.hidden, 96)
    want = ChunkedPrefill(LayerParams.from_arrays(shape, w)).prefill_chunk(x)
    stack = r.LayerStack(shape, [w], max_tokens=128, max_requests=1, max_pos=256, qkv_bias=True)
    for t in (33, 64, 100, 128):
        y = stack.prefill_batch(0, [stack.new_cache(t)], [t], r.to_device_bf16(x[:t]))
        check(f"{t} rows", r.to_numpy_f32(y), want[:t])


@functools.lru_cache(maxsize=1)
def _wide_layer():
    """A layer whose four matrices have 32 MB and more each, 127 rows, and what the oracle makes of them."""
    shape = synth.LayerShape("wide", 4352, 32, 4, 128, 4096)
    w = synth.layer_weights(shape, 103, qkv_bias=True, gains="uniform")
    x = synth.prompt_rows([("image", 127)], shape.hidden, 104)
    return shape, w, x, ChunkedPrefill(LayerParams.from_arrays(shape, w)).prefill_chunk(x)


@pytest.mark.parametrize("n_cu, splits", [(None, None), (None, "2"), ("128", "2"), ("128", "1"), ("64", "1"), ("40", "1")])
def test_tiles_of_streamed_weights(n_cu, splits, monkeypatch):
    """Every projection on tiles with the hint, in one block of rows: the compute-unit count and the K ranges steer the shape (QKV 64 x 64
    and with 64 and 40 units 128 x 96, 64 x 128 and 128 x 160; O and down cut along K on 64 x 64, 64 x 128, 128 x 64 and 128 x 128 and, in one
    range, on the same four).  Rows against the oracle, K and V (of 8-bit caches the codes) with the bits that the strips leave."""
    from paper_2509_24381_amd import runner as r
    shape, w, x, want = _wide_layer()
    xd = r.to_device_bf16(x)

    def calls(env):
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        stack = r.LayerStack(shape, [w], max_tokens=len(x), max_requests=1, max_pos=256, qkv_bias=True, fp8_visible_tokens=256)
        for k in env:
            monkeypatch.delenv(k)
        out = []
        for t in (61, 64, 96, 127):
            kv, kv8 = stack.new_cache(t), stack.new_cache_fp8(t, 0.0625, 0.0625)
            y = r.to_numpy_f32(stack.prefill_batch(0, [kv], [t], xd[:t]))
            stack.prefill_batch(0, [kv8], [t], xd[:t])
            out.append((t, y, [r.to_numpy_f32(c) for c in kv.export(0)] + [c.cpu().numpy() for c in kv8.export_codes(0)]))
        return out
    env = {k: v for k, v in (("RS_NCU", n_cu), ("RS_SPLITK", splits)) if v}
    for (t, y, tiles), (_, _, strips) in zip(calls(env), calls({**env, "RS_NARROW": "0"})):
        check(f"{t} rows", y, want[:t])
        for a, b in zip(tiles, strips):
            np.testing.assert_array_equal(a, b)
