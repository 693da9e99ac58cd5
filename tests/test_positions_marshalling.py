"""CPU: rotary positions reach the C ABI as the same ints whatever holds them and however it lies in memory."""
import numpy as np
import pytest
import torch

from paper_2509_24381_amd.binding import _positions_arg

BASE = np.arange(21).reshape(7, 3) * 5 % 97


@pytest.mark.parametrize("make", [
    lambda: BASE.tolist(), lambda: [tuple(r) for r in BASE], lambda: BASE.astype(np.int32), lambda: BASE.astype(np.int64),
    lambda: BASE.astype(np.uint8), lambda: np.asfortranarray(BASE.astype(np.int32)), lambda: np.repeat(BASE, 2, axis=0)[::2],
    lambda: np.ascontiguousarray(BASE[::-1, ::-1])[::-1, ::-1], lambda: BASE.astype(np.float32), lambda: BASE.astype(">i4"),
    lambda: torch.from_numpy(BASE), lambda: torch.from_numpy(BASE.T.copy()).T, lambda: torch.from_numpy(BASE).to(torch.float64),
    lambda: list(torch.from_numpy(BASE))])
def test_every_form_gives_the_same_ints(make):
    assert list(_positions_arg(make())) == BASE.flatten().tolist()


def test_values_beyond_an_int_wrap_as_before_and_no_rows_are_fine():
    assert list(_positions_arg(np.array([[2**32 + 5, -1, 2**31]]))) == list(_positions_arg([[2**32 + 5, -1, 2**31]]))
    for empty in ([], np.zeros((0, 3), dtype=np.int32), torch.zeros((0, 3), dtype=torch.int64)):
        assert len(_positions_arg(empty)) == 1
