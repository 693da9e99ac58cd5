"""GPU: the first kernel of a layer (norm factors, operand copy, the previous layer's pending sum): a workgroup per row in calls of few
rows, half a wavefront in others; rows whose chunks fill no pass."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 40, 250, 608, 609])
def test_a_stack_leaves_the_bits_of_its_layers(rows):
    """The sum of the down projection's K ranges inside the next layer's first kernel against the
    reduction kernel of its own: all layers in one call and one by one, bit for bit."""
    import torch
    from paper_2509_24381_amd import runner as r
    shape = synth.LayerShape("tiles", 192, 4, 2, 64, 16448)
    ws = [synth.layer_weights(shape, 93 + i, gains="uniform") for i in range(3)]
    stack = r.LayerStack(shape, ws, max_tokens=rows, max_requests=1, max_pos=2048)
    x = r.to_device_bf16(synth.prompt_rows([("image", rows)], 192, 94))
    kv_a, kv_b = stack.new_cache(rows), stack.new_cache(rows)
    y = x
    for layer in range(3):
        y = stack.prefill_batch(layer, [kv_a], [rows], y)
    z = torch.empty_like(x)
    stack.ctx.prefill_model_batch(stack.layers, [kv_b], [rows], x, z, stack.ctx.workspace(rows, 1))
    assert torch.equal(y.view(torch.int16), z.view(torch.int16))
    for layer in range(3):
        assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(kv_a.export(layer), kv_b.export(layer)))
