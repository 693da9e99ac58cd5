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
    call, which runs on tiles: the QKV projection accumulates along K in one order whatever the call's size."""
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


@pytest.mark.parametrize("hidden, inter, d", [(64, 64, 64), (320, 2112, 128), (1088, 320, 64)])
@pytest.mark.parametrize("by", [0, 1])
def test_packed_weights_are_the_rows_in_fragment_order(hidden, inter, d, by):
    """Every packed element against the layout written out in numpy, at widths of one slice of 256 features, of several and of a
    rest, and from sources that are only element-aligned where the call takes those (W_o and W_down): row t, features 8 c .. of
    a unit of 32 rows sit at chunk c, place t."""
    import ctypes as C
    import torch
    from paper_2509_24381_amd import runner as r
    from paper_2509_24381_amd.binding import _Weights, _check, _ptr
    hq, hkv = 4, 2
    ctx = r.Context(r.LayerConfig(hidden, hq, hkv, d, inter, qkv_bias=True, max_tokens_per_call=64, max_pos=64))
    rng = np.random.default_rng(hidden)
    q_dim, qkv = hq * d, (hq + 2 * hkv) * d
    g1, g2 = (synth.bf16_round(rng.uniform(0.5, 1.5, hidden).astype(np.float32)) for _ in range(2))
    mats = {"qkv": (qkv, hidden), "o": (hidden, q_dim), "gu": (2 * inter, hidden), "down": (hidden, inter)}
    mats = {k: synth.bf16_round(rng.standard_normal(s).astype(np.float32)) for k, s in mats.items()}

    def dev(a, shift=0):
        buf = torch.empty(a.size + shift, dtype=torch.bfloat16, device="cuda")
        buf[shift:].copy_(r.to_device_bf16(a).flatten())
        return buf[shift:]
    src = [dev(g1), dev(mats["qkv"]), dev(np.ones(qkv, np.float32)), dev(mats["o"], by), dev(g2), dev(mats["gu"]), dev(mats["down"], by)]
    slab = torch.empty(ctx.weights_packed_bytes(), dtype=torch.uint8, device="cuda")
    out, arg = _Weights(), _Weights(*[_ptr(t) for t in src])
    _check(ctx.lib.rs_weights_pack(ctx.handle, C.byref(arg), _ptr(slab), slab.numel(), C.byref(out), torch.cuda.current_stream().cuda_stream or None))

    def packed(ptr, rows, k):
        at = ptr - slab.data_ptr()
        return r.to_numpy_f32(slab[at: at + rows * k * 2].view(torch.bfloat16))

    def units(m, order):
        m = m[order]
        return m.reshape(m.shape[0] // 32, 32, m.shape[1] // 8, 8).transpose(0, 2, 1, 3).flatten()
    half = lambda base, n: [i for u in range(n // 16) for i in [*range(base + 16 * u, base + 16 * u + 16), *range(base + n + 16 * u, base + n + 16 * u + 16)]]
    qkv_order = [i for h in range(hq + hkv) for i in half(h * d, d // 2)] + list(range((hq + hkv) * d, qkv))
    names = [f[0] for f in _Weights._fields_]
    ptrs = {n: getattr(out, n) for n in names}
    for name, m, order, gain in (("w_qkv", mats["qkv"], qkv_order, g1), ("w_o", mats["o"], list(range(hidden)), None),
                                 ("w_gate_up", mats["gu"], half(0, inter), g2), ("w_down", mats["down"], list(range(hidden)), None)):
        want = m if gain is None else synth.bf16_round(m * gain)
        np.testing.assert_array_equal(packed(ptrs[name], *m.shape), units(want, order))
