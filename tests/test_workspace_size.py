"""CPU: how much workspace a call needs has a caller's static buffers behind it: calls that fitted 128 MiB keep fitting."""
import pytest

from paper_2509_24381_amd.binding import Context, LayerConfig


@pytest.mark.parametrize("dims, rows", [((3584, 28, 4, 128, 18944), 643), ((8192, 64, 8, 128, 29568), 317), ((8192, 64, 8, 128, 29568), 200)])
def test_calls_that_fit_the_static_workspace(dims, rows):
    h, hq, hkv, d, inter = dims
    ctx = Context(LayerConfig(hidden=h, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, mlp_inter=inter, max_tokens_per_call=1024, max_requests=1, max_pos=4096))
    assert ctx.lib.rs_workspace_bytes(ctx.handle, rows, 1) <= ctx.lib.rs_static_workspace_bytes()
