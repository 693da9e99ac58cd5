"""GPU: the projections of calls of 33 to 1024 rows (gemm_tile.h): every tile shape, row and unit counts that fill no tile, fewer steps of
64 k than the ring has slots, odd numbers of them, up to eight K ranges."""
import numpy as np
import pytest

import synth
from oracle import ChunkedPrefill, LayerParams
from test_gpu_parity import check

pytestmark = pytest.mark.gpu

ROWS = (33, 64, 65, 129, 200, 256, 257, 300, 511, 608, 609, 1024)


@pytest.mark.parametrize("n_cu", [None, "24", "80"])
@pytest.mark.parametrize("hidden, hq, hkv, d, inter", [(64, 2, 1, 64, 64), (320, 6, 2, 64, 2112), (192, 4, 2, 128, 8256), (1344, 10, 2, 128, 448)])
def test_tiles_against_the_oracle_and_the_strips(hidden, hq, hkv, d, inter, n_cu, monkeypatch):
    """Each row count against the oracle (bar of the layer, 1e-2), and K and V bit-identical to those that the strip kernel leaves (RS_NARROW=0)
    and to the same rows' of the longest call: all accumulate along K in one order.  The compute-unit count steers which shape and how many K ranges are chosen."""
    from paper_2509_24381_amd import runner as r
    shape = synth.LayerShape("tiles", hidden, hq, hkv, d, inter)
    w = synth.layer_weights(shape, 91, qkv_bias=True, gains="uniform")
    prior, longest = 70, max(ROWS)
    x = synth.prompt_rows([("text", prior), ("image", longest)], hidden, 92)
    st = ChunkedPrefill(LayerParams.from_arrays(shape, w))
    st.prefill_chunk(x[:prior])
    want = st.prefill_chunk(x[prior:])
    xd = r.to_device_bf16(x[prior:])

    def calls(**env):
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        stack = r.LayerStack(shape, [w], max_tokens=longest, max_requests=1, max_pos=2048, qkv_bias=True)
        for k in env:
            monkeypatch.delenv(k)
        kv = stack.new_cache(prior + longest)
        stack.prefill_batch(0, [kv], [prior], r.to_device_bf16(x[:prior]))
        out = []
        for t in ROWS:
            kv.truncate(0, prior)
            y = r.to_numpy_f32(stack.prefill_batch(0, [kv], [t], xd[:t]))
            out.append((y, *(r.to_numpy_f32(c) for c in kv.export(0))))
        return out
    env = {} if n_cu is None else {"RS_NCU": n_cu}
    of_tiles = calls(**env)
    longest_call = of_tiles[-1]
    for t, tiles, strips in zip(ROWS, of_tiles, calls(RS_NARROW="0", **env)):
        check(f"{t} rows of H={hidden} I={inter}", tiles[0], want[:t])
        np.testing.assert_array_equal(tiles[1], strips[1])
        np.testing.assert_array_equal(tiles[2], strips[2])
        np.testing.assert_array_equal(tiles[1], longest_call[1][:prior + t])
        np.testing.assert_array_equal(tiles[2], longest_call[2][:prior + t])


@pytest.mark.parametrize("lens", [(1, 2, 27), (63, 65, 130, 1), (200, 7, 500, 317)])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_caches_that_the_projection_fills(d, paged, lens, monkeypatch):
    """Several requests at once: the projection's epilogue and the first kernel's zeros leave every byte of the caches' slabs as the append
    kernel (RS_NARROW=0) does, from slabs that start as NaN patterns, at first rows inside, at the start and at the end of a block of
    64 tokens."""
    import torch
    from paper_2509_24381_amd import runner as r
    priors = (0, 61, 64, 130)[:len(lens)]
    shape = synth.LayerShape("append", 192, 4, 2, d, 448)
    w = synth.layer_weights(shape, 105, qkv_bias=True, gains="uniform")
    x = r.to_device_bf16(synth.prompt_rows([("image", sum(lens))], shape.hidden, 106))

    def run():
        stack = r.LayerStack(shape, [w], max_tokens=1024, max_requests=4, max_pos=2048, qkv_bias=True)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(107)
        pool = stack.new_pool(40) if paged else None
        kvs = [pool.new_cache(1) if paged else stack.new_cache(p + n) for p, n in zip(priors, lens)]
        slabs = [pool.slab] if paged else [kv.slab for kv in kvs]
        for s in slabs:
            s.view(torch.int16).fill_(0x7FC1)
        for kv, p in zip(kvs, priors):
            if p:
                k, v = (torch.randn(p, 2, d, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
                kv.import_(0, k, v)
        y = stack.prefill_batch(0, kvs, list(lens), x)
        return y, slabs
    y, slabs = run()
    monkeypatch.setenv("RS_NARROW", "0")
    want_y, want = run()
    check("rows", r.to_numpy_f32(y), r.to_numpy_f32(want_y))
    for a, b in zip(slabs, want):
        assert torch.equal(a, b)
