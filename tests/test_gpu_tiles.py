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
