"""GPU: calls of few rows (gemm_skinny.h) at the edges of its rules: 32, 64 and 128 rows, K ranges that leave wavefronts with
different numbers of k-steps, K long enough for eight wavefronts and for two K ranges, layers too wide for the rules."""
import numpy as np
import pytest

import synth
from oracle import ChunkedPrefill, LayerParams
from test_gpu_parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden, inter, d", [(64, 64, 64), (192, 4096, 128), (128, 8256, 64), (1088, 320, 128), (2304, 1024, 64)])
def test_few_rows_against_the_oracle_and_a_longer_call(hidden, inter, d):
    """Each row count against the oracle (bar of the layer, 1e-2), and K and V bit-identical to the same rows' of a 300-row
    call, which runs in the strip kernel: the QKV projection accumulates along K in one order whatever the call's size."""
    from paper_2509_24381_amd import runner as r
    shape = synth.LayerShape("few", hidden, 4, 2, d, inter)
    w = synth.layer_weights(shape, 88, qkv_bias=True, gains="uniform")
    stack = r.LayerStack(shape, [w], max_tokens=320, max_requests=1, max_pos=1024, qkv_bias=True)
    prior, longest = 70, 300
    x = synth.prompt_rows([("text", prior), ("image", longest)], hidden, 89)
    st = ChunkedPrefill(LayerParams.from_arrays(shape, w))
    st.prefill_chunk(x[:prior])
    want = st.prefill_chunk(x[prior:])
    kv = stack.new_cache(prior + longest)
    stack.prefill_batch(0, [kv], [prior], r.to_device_bf16(x[:prior]))
    xd = r.to_device_bf16(x[prior:])
    check("300 rows", r.to_numpy_f32(stack.prefill_batch(0, [kv], [longest], xd)), want)
    k_long, v_long = (r.to_numpy_f32(t) for t in kv.export(0))
    for t in (1, 31, 32, 33, 64, 65, 113, 114, 127, 128, 129):
        kv.truncate(0, prior)
        y = r.to_numpy_f32(stack.prefill_batch(0, [kv], [t], xd[:t]))
        check(f"{t} rows of H={hidden} I={inter}", y, want[:t])
        k, v = (r.to_numpy_f32(c) for c in kv.export(0))
        np.testing.assert_array_equal(k, k_long[:prior + t])
        np.testing.assert_array_equal(v, v_long[:prior + t])
