"""Sequence lengths reach the library the same whatever container they come in."""
import ctypes

import numpy as np
import pytest


@pytest.mark.parametrize("form", [lambda x: x, tuple, lambda x: np.array(x), lambda x: np.array(x, dtype=np.int32), lambda x: [np.int64(v) for v in x],
                                  lambda x: np.repeat(np.array(x), 2)[::2]])
@pytest.mark.parametrize("lens", [[5], [], [33, 131072, 4115], [0, -3, (1 << 31) - 1]])
def test_lengths(form, lens):
    from paper_2509_09754_amd import lava
    arr, n, total = lava._lengths(form(list(lens)))
    assert isinstance(arr, ctypes.Array) and arr._type_ is ctypes.c_int64
    want = np.asarray(form(list(lens))).astype(np.int64)
    assert list(arr) == want.tolist() and n == len(lens) and total == int(want.sum())
