"""GPU: projections whose weights are loaded with the streaming hint."""
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
