"""GPU: the first kernel of a layer (norm factors, operand copy, the previous layer's pending sum): a workgroup per row in calls of few
rows, half a wavefront in others; rows whose chunks fill no pass."""
import numpy as np
import pytest

import synth
from oracle import LayerParams, layer_forward
from test_gpu_parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden", [192, 2112, 4352])
def test_keys_and_values_do_not_depend_on_the_form(hidden):
    """K and V of the same rows, bit for bit, from calls of every form: a workgroup per row (up to 608 rows), half a wavefront (609 and
    more), and the projection's own forms up to strips of more than 1024 rows.  192 features fill 24 of a row's 256 places; 2112 and 4352
    reach the second pass of half a wavefront and of a workgroup, and end in the middle of one.  The longest call against the oracle."""
    from paper_2509_24381_amd import runner as r
    shape = synth.LayerShape("forms", hidden, 2, 1, 64, 64)
    w = synth.layer_weights(shape, 101, qkv_bias=True, gains="uniform")
    calls = (33, 256, 607, 608, 609, 1024, 1030)
    x = synth.prompt_rows([("text", 200), ("image", max(calls) - 200)], hidden, 102)
    stack = r.LayerStack(shape, [w], max_tokens=max(calls), max_requests=1, max_pos=2048, qkv_bias=True)
    xd = r.to_device_bf16(x)

    def leave(rows):
        kv = stack.new_cache(rows)
        stack.prefill_batch(0, [kv], [rows], xd[:rows])
        return [r.to_numpy_f32(t) for t in kv.export(0)]
    k, v = leave(calls[-1])
    _, k_ref, v_ref = layer_forward(x, LayerParams.from_arrays(shape, w))
    check("K", k, k_ref)
    check("V", v, v_ref)
    for rows in calls[:-1]:
        got_k, got_v = leave(rows)
        np.testing.assert_array_equal(got_k, k[:rows])
        np.testing.assert_array_equal(got_v, v[:rows])


@pytest.mark.parametrize("rows", [1, 40, 250, 608, 609])
@pytest.mark.parametrize("hidden, inter, splits", [(192, 16448, None), (4352, 1024, "4")])
def test_a_stack_leaves_the_bits_of_its_layers(hidden, inter, splits, rows, monkeypatch):
    """The sum of the down projection's K ranges inside the next layer's first kernel against the
    reduction kernel of its own: all layers in one call and one by one, bit for bit.  192 features: up to eight ranges; 4352: a second
    pass over the row in both forms."""
    import torch
    from paper_2509_24381_amd import runner as r
    if splits:
        monkeypatch.setenv("RS_SPLITK", splits)
    shape = synth.LayerShape("tiles", hidden, 4, 2, 64, inter)
    ws = [synth.layer_weights(shape, 93 + i, gains="uniform") for i in range(3)]
    stack = r.LayerStack(shape, ws, max_tokens=rows, max_requests=1, max_pos=2048)
    x = r.to_device_bf16(synth.prompt_rows([("image", rows)], hidden, 94))
    kv_a, kv_b = stack.new_cache(rows), stack.new_cache(rows)
    y = x
    for layer in range(3):
        y = stack.prefill_batch(layer, [kv_a], [rows], y)
    z = torch.empty_like(x)
    stack.ctx.prefill_model_batch(stack.layers, [kv_b], [rows], x, z, stack.ctx.workspace(rows, 1))
    assert torch.equal(y.view(torch.int16), z.view(torch.int16))
    for layer in range(3):
        assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(kv_a.export(layer), kv_b.export(layer)))
