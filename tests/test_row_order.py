"""The order in which a decode call's row kernels take its rows, on the host: every row once, with its own model."""
import numpy as np
import pytest

from paper_2603_13281_amd import binding


@pytest.mark.parametrize("last", [0, 7, 32765, 32766, 32767, 32768, 65534, 65535, 65536, 2 ** 31 - 1])
@pytest.mark.parametrize("rows", [1, 96, 97, 120, 316, 65535])
def test_every_row_once_with_its_model(rows, last):
    model = np.arange(rows, dtype=np.int64) % 3 - 1
    model[model == 1] = last                                       # encoder rows, model 0 and the call's largest id
    entries = binding.row_order(model)
    assert len(entries) <= rows + 16 and len(entries) % 8 == 0
    if len(entries) == 0:                                          # the kernels then read each row's model themselves
        return
    taken = entries[entries >= 0].astype(np.int64)
    np.testing.assert_array_equal(np.sort(taken & 0xffff), np.arange(rows))
    np.testing.assert_array_equal((taken >> 16) - 1, model[taken & 0xffff])
