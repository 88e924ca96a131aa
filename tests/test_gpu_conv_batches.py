"""The conv forward's record batches at every length: event rows that hold
exactly 0, 1, ..., 17 records (one batch of 8 holds 1 to 8 of them, partial
batches take their own branch), in the chunked walk (more than 32 channels), in
its second channel tile and in the list form (two positions per wave whose rows
differ in length). Against the oracle with the error model of the conv tests."""
import numpy as np
import pytest

from tests.test_gpu_conv import _conv_case, _conv_parity, _cs, dev  # noqa: F401

pytestmark = pytest.mark.gpu

ROWS = 18  # rows of 0 .. 17 records: 153 inputs of a 1 x 1 receptive field


@pytest.mark.parametrize("c_out,silent", [(64, 0), (70, 0), (20, 0), (32, 5)])
def test_rows_of_every_length(dev, c_out, silent):  # noqa: F811
    n = ROWS * (ROWS - 1) // 2
    cs = _cs(n, 2, 3, c_out, K=1, pad=0)
    p, t, W = _conv_case(31, 2, cs, ROWS + 2, 1.0, 0.3, k=7.0)
    rng = np.random.default_rng(32)
    for b in range(t.shape[0]):
        for y in range(2):
            for x in range(3):
                # the row that holds k records differs from position to position
                row = np.repeat(rng.permutation(ROWS), np.arange(ROWS))
                v = (row + 0.2 + 0.6 * rng.random(n)) * p["dt"]
                v[rng.choice(n, silent, replace=False)] = np.inf
                t[b, :, y, x] = rng.permutation(v)
    _conv_parity(dev, p, cs, t, W, f"rows of 0..17 records, {c_out} channels")
