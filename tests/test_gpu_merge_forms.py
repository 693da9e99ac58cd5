"""GPU: the forms of the merge of split key ranges: up to four parts, more in a launch that is resident at once, and more in a larger one
(RS_NCU stands in for the device's size)."""
import pytest

import synth
from oracle import ChunkedPrefill, LayerParams
from test_gpu_parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("parts, n_cu", [("2", None), ("4", "2"), ("5", None), ("5", "2"), ("16", None), ("16", "2")])
def test_merge_forms_against_the_oracle(parts, n_cu, d, monkeypatch):
    from paper_2509_24381_amd import runner as r
    monkeypatch.setenv("RS_ATTN_SPLIT", parts)
    if n_cu:
        monkeypatch.setenv("RS_NCU", n_cu)
    shape = synth.LayerShape("merge", 128, 4, 2, d, 192)
    w = synth.layer_weights(shape, 97, gains="uniform")
    prior, rows = 6400, 140
    x = synth.prompt_rows([("text", prior), ("image", rows)], shape.hidden, 98)
    st = ChunkedPrefill(LayerParams.from_arrays(shape, w))
    st.prefill_chunk(x[:prior])
    want = st.prefill_chunk(x[prior:])
    stack = r.LayerStack(shape, [w], max_tokens=prior, max_requests=1, max_pos=8192)
    kv = stack.new_cache(prior + rows)
    stack.prefill_batch(0, [kv], [prior], r.to_device_bf16(x[:prior]))
    y = r.to_numpy_f32(stack.prefill_batch(0, [kv], [rows], r.to_device_bf16(x[prior:])))
    check(f"{parts} parts", y, want)
