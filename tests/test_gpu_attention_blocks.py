"""GPU: the attention kernel where its blocks, tiles and parts end, and where its reference maximum has to move.

Attention is isolated by a zero down projection (y = x + attention W_o^T).  The attention term carries the bfloat16
roundings of q, k, v, the probabilities, the output and y (2^-9 / sqrt(3) = 1.1e-3 to 1.7e-3 each, six of them in quadrature
about 4e-3, twice that where y is dominated by x): 2e-2 leaves a factor of two to three.
"""
import numpy as np
import pytest

import synth
from test_gpu_parity import check, oracle_batch, run_batch

pytestmark = pytest.mark.gpu


def _requests(shape, spec, seed, key_scale=None):
    rng = np.random.default_rng(seed)
    reqs = []
    for prior, t_new in spec:
        pk = rng.standard_normal((prior, shape.n_kv_heads, shape.head_dim), dtype=np.float32)
        if key_scale is not None:
            pk = pk * key_scale(prior)[:, None, None]
        pv = rng.standard_normal((prior, shape.n_kv_heads, shape.head_dim), dtype=np.float32)
        rows = synth.prompt_rows([("text", t_new)], shape.hidden, seed + 1 + len(reqs))
        reqs.append(synth.BatchRequest(prior, synth.bf16_round(pk), synth.bf16_round(pv), rows))
    return reqs


def _attention_term(shape, reqs, name, tol, capacity):
    w = synth.layer_weights(shape, 41, gains="uniform")
    w.wd = np.zeros_like(w.wd)
    y, _ = run_batch(shape, w, reqs, capacity=capacity)
    y_ref, _ = oracle_batch(shape, w, reqs)
    x = np.concatenate([r.rows for r in reqs], axis=0)
    off = 0
    for i, r in enumerate(reqs):
        n = r.rows.shape[0]
        check(f"{name}, request {i}", (y - x)[off: off + n], (y_ref - x)[off: off + n], tol=tol)
        off += n


# (blocks of 256 rows with eight wavefronts run in calls of more than two small blocks per compute unit with a walk of more than 64
# tiles: planned for one unit, the second request makes that of all of these; without it they run blocks of 128 rows with four)
LONG = (4200, 40)
@pytest.mark.parametrize("n_cu", [None, "1"])
@pytest.mark.parametrize("heads", [(4, 4, 64), (7, 1, 128), (8, 1, 64), (2, 2, 128)])
@pytest.mark.parametrize("prior, t_new", [(0, 1), (0, 31), (0, 33), (0, 64), (31, 32), (32, 33), (63, 1), (64, 36), (65, 37),
                                          (100, 255), (127, 256), (129, 257)])
def test_ends_of_half_tiles_tiles_and_blocks(heads, prior, t_new, n_cu, monkeypatch):
    """Rows and keys that end just before, at and behind a half tile (32 keys), a tile (64), a wavefront's 32 stacked rows and
    a block's 128 or 256, with 1, 7 and 8 query heads per KV head (256 rows are then 256, 37 and 32 tokens)."""
    if n_cu:
        monkeypatch.setenv("RS_NCU", n_cu)
    hq, hkv, d = heads
    shape = synth.LayerShape("edge", 256, hq, hkv, d, 256)
    spec = [(prior, t_new)] + ([LONG] if n_cu else [])
    _attention_term(shape, _requests(shape, spec, 500 + prior), f"{heads} P={prior} T={t_new}", 2e-2, 4352)


@pytest.mark.parametrize("n_cu", [None, "1"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("at", [(31,), (32,), (45,), (64, 100), (63, 159, 160, 255), (77, 109, 130, 150, 200, 229)])
def test_scores_that_jump_inside_a_tile(d, at, n_cu, monkeypatch):
    """Single keys whose scores stand far above all before them (by up to 2^25 in the probabilities), in the first and in the
    second half of a tile: the reference has to move at that half, for the queries concerned, without touching the half that is
    still to be multiplied (keys of the first tile only raise where it starts).  Sharp distributions turn the absolute score error (2.4e-3 of a score of about 15) into the
    weights: 4e-2."""
    if n_cu:
        monkeypatch.setenv("RS_NCU", n_cu)
    shape = synth.LayerShape("jump", 256, 4, 2, d, 256)

    def scale(prior):
        s = np.ones(prior, dtype=np.float32)
        s[list(at)] = 14.0
        return s
    spec = [(300, 90)] + ([LONG] if n_cu else [])
    _attention_term(shape, _requests(shape, spec, 600 + at[0], scale), f"d={d} jumps at {at}", 4e-2, 4352)


@pytest.mark.parametrize("n_cu", ["3", "7", "12", "40", "300"])
def test_key_ranges_cut_for_unequal_requests(n_cu, monkeypatch):
    """Requests with caches of very different lengths in one call, planned for different compute-unit counts: nothing cut,
    equal parts, and parts of an even share with a rest, in blocks of eight and of four wavefronts."""
    monkeypatch.setenv("RS_NCU", n_cu)
    shape = synth.LayerShape("small128", 256, 4, 2, 128, 256)
    spec = [(5000, 40), (0, 70), (900, 33), (1500, 128), (64, 1), (2047, 129)]
    _attention_term(shape, _requests(shape, spec, 700), f"planned for {n_cu} units", 2e-2, 5120)


@pytest.mark.parametrize("n_cu, split, prior, t_new", [(None, None, 900, 30), ("1", None, 4200, 200), (None, "2", 900, 30)])
@pytest.mark.parametrize("d", [64, 128])
def test_keys_that_score_minus_infinity(d, n_cu, split, prior, t_new, monkeypatch):
    """Cached keys whose score is minus infinity for every query weigh nothing, also where they are the first 32 keys of a
    cache or of a part, the first 64 (those the reference starts from), and a whole later half tile."""
    for name, value in (("RS_NCU", n_cu), ("RS_ATTN_SPLIT", split)):
        if value:
            monkeypatch.setenv(name, value)
    shape = synth.LayerShape("minf", 256, 4, 2, d, 256)
    reqs = _requests(shape, [(prior, t_new)], 800)
    for first in (0, 7 * 64, 600):    # (15 tiles in two parts: the second starts at tile 7)
        reqs[0].prior_k[first: first + (64 if first == 0 else 32), :, d // 2 - 1] = -np.inf
    # q is its bias alone; its slowest rotary pair is (1, 1), which the rotation at these positions leaves positive
    w = synth.layer_weights(shape, 41, qkv_bias=True, gains="uniform")
    w.wq, w.wd = np.zeros_like(w.wq), np.zeros_like(w.wd)
    bq = w.bq.reshape(shape.n_q_heads, d)
    bq[:, [d // 2 - 1, d - 1]] = 1.0
    y, y_ref = _run_with_bias(shape, w, reqs, 4416)
    check(f"d={d} keys at minus infinity", y - reqs[0].rows, y_ref - reqs[0].rows, tol=2e-2)


def _run_with_bias(shape, w, reqs, capacity):
    from paper_2509_24381_amd import runner as r
    stack = r.LayerStack(shape, [w], max_tokens=256, max_requests=1, max_pos=capacity, qkv_bias=True)
    kv = stack.new_cache(capacity)
    kv.import_(0, r.to_device_bf16(reqs[0].prior_k), r.to_device_bf16(reqs[0].prior_v))
    y = r.to_numpy_f32(stack.prefill_batch(0, [kv], [reqs[0].rows.shape[0]], r.to_device_bf16(reqs[0].rows)))
    return y, oracle_batch(shape, w, reqs)[0]


def test_layers_of_different_lengths_in_one_call():
    """The layers of one call whose caches are equally long share one plan; where the lengths change, so must the plan: the same
    bits as layer by layer, with caches cut into parts, too short for that, and long again."""
    import torch
    from paper_2509_24381_amd import runner as r
    shape = synth.LayerShape("lens", 256, 4, 2, 128, 256)
    w = synth.layer_weights(shape, 42, gains="uniform")
    stack = r.LayerStack(shape, [w] * 4, max_tokens=80, max_requests=2, max_pos=3200)
    lens, priors = [50, 30], [[2000, 2000, 300, 2500], [100, 100, 100, 900]]
    rng = np.random.default_rng(43)
    x = r.to_device_bf16(synth.prompt_rows([("text", sum(lens))], shape.hidden, 44))
    made = [[[r.to_device_bf16(rng.standard_normal((p, 2, 128), dtype=np.float32)) for _ in range(2)] for p in ps] for ps in priors]

    def caches():
        kvs = [stack.new_cache(2600) for _ in lens]
        for kv, layers in zip(kvs, made):
            for l, (k, v) in enumerate(layers):
                kv.import_(l, k, v)
        return kvs
    a, b = caches(), caches()
    y = torch.empty_like(x)
    stack.ctx.prefill_model_batch(stack.layers, a, lens, x, y, stack.ws)
    z = x
    for l in range(4):
        z = stack.prefill_batch(l, b, lens, z)
    assert torch.equal(y.view(torch.int16), z.view(torch.int16))
    for kv_a, kv_b in zip(a, b):
        for l in range(4):
            assert all(torch.equal(s.view(torch.int16), t.view(torch.int16)) for s, t in zip(kv_a.export(l), kv_b.export(l)))
