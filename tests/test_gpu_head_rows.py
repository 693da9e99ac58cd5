"""GPU: the first-token head's matrix path (3 rows and more) at the edges of its groups, shares and K ranges, against the
oracle, and where it must hand over to plain fp32 arithmetic.

Both kernels keep the rows' values to fp32 or better and sum in fp32: the error against 64 bits is 1.0e-7 to 1.5e-7 measured on
3584 and 8192 features (2-norm); 1e-6 leaves a margin for small vocabularies.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import synth
from oracle import first_token_logits, rel_fro

pytestmark = pytest.mark.gpu


def _head(hidden, vocab, n_rows, seed=71):
    from paper_2509_24381_amd import runner
    shape = synth.LayerShape("lm", hidden, 2, 1, 64, 64)
    ctx = runner.Context(runner.config_for(shape, max_tokens=32, max_requests=1, max_pos=64))
    rng = np.random.default_rng(seed)
    g = synth.bf16_round(rng.uniform(0.5, 1.5, hidden).astype(np.float32))
    w = synth.bf16_round((rng.standard_normal((vocab, hidden)) * 0.02).astype(np.float32))
    x = synth.bf16_round(rng.standard_normal((n_rows, hidden)).astype(np.float32))
    return runner, ctx, shape, g, w, x


@pytest.mark.parametrize("hidden, vocab, n_rows", [(64, 64, 3), (128, 63, 4), (192, 65, 10), (256, 1, 11), (320, 16385, 20),
                                                   (704, 5000, 21), (3584, 777, 41), (8192, 300, 9)])
def test_logits_of_three_rows_and_more(hidden, vocab, n_rows):
    """One to eleven groups of 64 features for four wavefronts (some without any), vocabularies of one row, of a tile and one
    more or less, and of a share with a remainder; one and two groups of rows, and passes of 20 with a rest."""
    runner, ctx, shape, g, w, x = _head(hidden, vocab, n_rows)
    got = ctx.lm_head(runner.to_device_bf16(g), runner.to_device_bf16(w), runner.to_device_bf16(x)).cpu().numpy()
    err = rel_fro(got, first_token_logits(x, g, w, shape.rms_eps))
    print(f"[parity] logits H={hidden} V={vocab} R={n_rows}: {err:.2e}", flush=True)
    assert err <= 1e-6


def test_a_row_has_the_same_logits_in_every_call_of_three_rows_and_more():
    """One and two groups of rows, passes with a rest, first and last places: bit for bit."""
    runner, ctx, shape, g, w, x = _head(704, 3000, 23)
    gd, wd, xd = (runner.to_device_bf16(a) for a in (g, w, x))
    all_rows = ctx.lm_head(gd, wd, xd)
    for first, n in ((0, 3), (5, 9), (2, 10), (0, 11), (3, 20), (19, 4)):
        assert torch.equal(ctx.lm_head(gd, wd, xd[first: first + n].contiguous()), all_rows[first: first + n])


@pytest.mark.parametrize("n_rows", [1, 2, 3, 10, 11, 21])
def test_a_vocabulary_that_is_streamed(n_rows):
    """Vocabularies of 256 MiB and more are loaded with the streaming hint: every logit has the bits that a call on a part of the
    vocabulary below that size gives, in either kernel, and sampled words (first, last, and across the parts' border) meet the oracle."""
    from paper_2509_24381_amd import runner
    hidden, vocab, part = 1024, 131201, 70001
    shape = synth.LayerShape("lm", hidden, 2, 1, 64, 64)
    ctx = runner.Context(runner.config_for(shape, max_tokens=32, max_requests=1, max_pos=64))
    assert part * hidden * 2 < 1 << 28 <= vocab * hidden * 2
    rng = np.random.default_rng(73)
    g = synth.bf16_round(rng.uniform(0.5, 1.5, hidden).astype(np.float32))
    x = synth.bf16_round(rng.standard_normal((n_rows, hidden)).astype(np.float32))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(74)
    wd = (torch.randn(vocab, hidden, device="cuda", generator=gen) * 0.02).to(torch.bfloat16)
    gd, xd = runner.to_device_bf16(g), runner.to_device_bf16(x)
    got = ctx.lm_head(gd, wd, xd)
    for first, end in ((0, part), (part, vocab)):
        assert torch.equal(got[:, first:end], ctx.lm_head(gd, wd[first:end].contiguous(), xd))
    words = np.unique(np.concatenate([[0, 1, part - 1, part, vocab - 2, vocab - 1], rng.integers(0, vocab, 500)]))
    want = first_token_logits(x, g, runner.to_numpy_f32(wd[torch.from_numpy(words).cuda()]), shape.rms_eps)
    assert rel_fro(got[:, torch.from_numpy(words).cuda()].cpu().numpy(), want) <= 1e-6


def test_a_workspace_of_four_bytes_per_value_is_still_enough():
    """4 H bytes per row (rounded up to 256) is all the fp32 kernel needs; the same call with the full size takes the matrix
    path.  Both meet the bar; a smaller workspace is refused."""
    runner, ctx, shape, g, w, x = _head(1024, 3000, 5)
    gd, wd, xd = (runner.to_device_bf16(a) for a in (g, w, x))
    out = torch.empty((5, 3000), dtype=torch.float32, device="cuda")
    ws = torch.empty(ctx.lib.rs_lm_head_workspace_bytes(ctx.handle, 5), dtype=torch.uint8, device="cuda")
    want = first_token_logits(x, g, w, shape.rms_eps)
    for n, ok in [(5 * 1024 * 4, True), (ws.numel(), True), (5 * 1024 * 4 - 256, False)]:
        out.fill_(0)
        st = ctx.lib.rs_lm_head(ctx.handle, gd.data_ptr(), wd.data_ptr(), 3000, xd.data_ptr(), 5, out.data_ptr(), ws.data_ptr(),
                                C.c_size_t(n), torch.cuda.current_stream().cuda_stream or None)
        assert st == (0 if ok else -3)
        if ok:
            assert rel_fro(out.cpu().numpy(), want) <= 1e-6


def test_infinite_weights_and_nan_rows_stay_where_they_are():
    """An infinite weight gives infinite logits of h's sign in its vocabulary row only; a row of x with a NaN gives NaN in
    that row only."""
    runner, ctx, shape, g, w, x = _head(256, 200, 6)
    w[17, 5], w[130, 200] = np.inf, -np.inf
    x[2, 9] = np.nan
    got = ctx.lm_head(runner.to_device_bf16(g), runner.to_device_bf16(w), runner.to_device_bf16(x)).cpu().numpy()
    rows = [0, 1, 3, 4, 5]
    assert np.all(np.isnan(got[2]))
    np.testing.assert_array_equal(got[rows, 17], np.where(x[rows, 5] > 0, np.inf, -np.inf))
    np.testing.assert_array_equal(got[rows, 130], np.where(x[rows, 200] > 0, -np.inf, np.inf))
    fin = np.delete(np.arange(200), [17, 130])
    want = first_token_logits(x[rows], g, w[fin], shape.rms_eps)
    assert rel_fro(got[np.ix_(rows, fin)], want) <= 1e-6


def _call_with_workspace(ctx, g, w, x):
    """Logits and the bytes the call left in its workspace."""
    n, vocab = int(x.shape[0]), int(w.shape[0])
    out = torch.empty((n, vocab), dtype=torch.float32, device="cuda")
    ws = torch.zeros(ctx.lib.rs_lm_head_workspace_bytes(ctx.handle, n), dtype=torch.uint8, device="cuda")
    assert ctx.lib.rs_lm_head(ctx.handle, g.data_ptr(), w.data_ptr(), vocab, x.data_ptr(), n, out.data_ptr(), ws.data_ptr(),
                              C.c_size_t(ws.numel()), torch.cuda.current_stream().cuda_stream or None) == 0
    return out.cpu().numpy(), ws


@pytest.mark.parametrize("hidden", [64, 3584])
def test_the_three_pieces_sum_to_the_normalised_value(hidden):
    """What the matrix path leaves in its workspace - three bfloat16 pieces per normalised value, columns 10 s + r of a group
    of 10 rows - sums to u g within 2^-26, u = x / rms being the fp32 row that a call of one row with gains of one leaves
    there.  (hi is within 2^-9 of the product, mid within 2^-9 of the difference and lo within 2^-9 of the next: 2^-27.)  One
    gain is the largest bfloat16 number: its product rounds to an infinite bfloat16 where the fp32 value is still finite."""
    runner, ctx, shape, g, w, x = _head(hidden, 64, 13)
    g[7] = synth.bf16_round(np.array([3.3895314e38], dtype=np.float32))[0]
    x[:, 7] = 1.0     # h = g / rms(x), finite where the rms is not below 1
    x[0] = np.where(np.arange(hidden) % 2 == 0, 1.0, -1.0)
    x[0, np.arange(hidden) % 4 != 3] *= 0.99609375     # an rms of 0.997: h lies between the two largest values
    gd, wd, xd, ones = (runner.to_device_bf16(a) for a in (g, w, x, np.ones_like(g)))
    _, ws = _call_with_workspace(ctx, gd, wd, xd)
    pieces = ws[: 2 * (hidden // 16) * 512 * 2].view(torch.bfloat16).double().cpu().numpy()
    pieces = pieces.reshape(2, hidden // 16, 2, 32, 8).transpose(0, 3, 1, 2, 4).reshape(2, 32, hidden)
    edge = 0
    for r in range(13):
        _, ws1 = _call_with_workspace(ctx, ones, wd, xd[r:r + 1])
        with np.errstate(over='ignore'):
            want = ws1[: hidden * 4].view(torch.float32).double().cpu().numpy() * g.astype(np.float64)
        keep = np.abs(want) <= np.finfo(np.float32).max
        edge += int(np.sum(keep & (np.abs(want) > 3.3961e38)))
        got = sum(pieces[r // 10, 10 * s + r % 10][keep] for s in range(3))
        assert np.all(np.abs(got - want[keep]) <= 2.0 ** -26 * np.abs(want)[keep])
    assert edge > 0, "no value between the largest bfloat16 and the largest fp32 number"


def test_infinite_gains_give_the_logits_of_the_fp32_path():
    """An infinite gain makes one normalised value infinite, or NaN where x is zero: infinite logits of its sign, NaN beside a zero
    weight, and what infinite weights make of it - in calls of six rows as in calls of one, which take the fp32 kernel."""
    runner, ctx, shape, g, w, x = _head(256, 200, 6)
    g[5] = np.inf
    x[4, 5] = 0.0
    w[3, 5] = 0.0
    w[17, 9], w[130, 200], w[131, 5] = np.inf, -np.inf, -np.inf
    gd, wd, xd = (runner.to_device_bf16(a) for a in (g, w, x))
    got = ctx.lm_head(gd, wd, xd).cpu().numpy()
    for r in range(6):
        np.testing.assert_array_equal(got[r:r + 1], ctx.lm_head(gd, wd, xd[r:r + 1]).cpu().numpy())   # (nothing is finite)
    assert np.all(np.isnan(got[4])) and np.all(np.isnan(got[:, 3])) and np.isinf(got[0]).sum() >= 197


def test_an_infinite_activation_costs_no_more_than_any_other():
    """A row of x with an infinity away from feature 0 (its normalised values are zeros and one NaN) gives NaN logits in the
    time of an ordinary call: nothing is worked out again logit by logit.  (Factor 3 between medians of five: walking every
    logit's row once more took well over ten times the call.)"""
    runner, ctx, shape, g, w, x = _head(3584, 16000, 6)
    bad = x.copy()
    bad[2, 1000] = np.inf
    gd, wd, xd, bd = (runner.to_device_bf16(a) for a in (g, w, x, bad))

    def median_ms(rows):
        ts = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            out = ctx.lm_head(gd, wd, rows)
            b.record()
            torch.cuda.synchronize()
            ts.append(a.elapsed_time(b))
        return sorted(ts[1:])[2], out
    t_plain, plain = median_ms(xd)
    t_bad, out = median_ms(bd)
    print(f"[head] plain {t_plain * 1e3:.0f} us, with an infinite activation {t_bad * 1e3:.0f} us", flush=True)
    keep = [0, 1, 3, 4, 5]
    assert bool(torch.isnan(out[2]).all()) and torch.equal(out[keep], plain[keep])
    assert t_bad <= 3 * t_plain
