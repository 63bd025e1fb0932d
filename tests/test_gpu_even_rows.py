"""SpMM where rows are long: windows that one row fills, and even rows of medium length, which have a kernel of their own; at
the lengths where the choice changes, with a row that is longer than the others by just as much as still counts as even, rows
without entries, widths with and without 16-byte pieces, and a row that crosses more than 64 windows.  Against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_04305_amd as sp
from gen import prng
from gpu_util import say, dev, gpu_pack, assert_product_close, DEV

pytestmark = pytest.mark.gpu


def matrix(lens, n, dtype):
    """A row of lens[i] entries for every i, spread over n columns."""
    lens = np.asarray(lens, dtype=np.int64)
    rows = np.repeat(np.arange(lens.size, dtype=np.int64), lens)
    at = np.arange(rows.size, dtype=np.int64) - np.repeat(np.cumsum(lens) - lens, lens)
    cols = at * (n // np.maximum(np.repeat(lens, lens), 1))
    return rows, cols, prng.uniform_pm1(11, 1, rows.size, dtype=dtype)


def check(lens, n, dtype, widths, what, lt=(0, 1)):
    rows, cols, vals = matrix(lens, n, dtype)
    A = gpu_pack(lt, (0, 1), (len(lens), n), [rows, cols], vals)
    for N in widths:
        B = prng.uniform_pm1(11, 2, n * N, dtype=dtype).reshape(-1, N)
        C0 = prng.uniform_pm1(11, 3, len(lens) * N, dtype=dtype).reshape(-1, N)
        ref, mag = oracle.matmul_coo((len(lens), n), rows, cols, vals, B)
        for accumulate in (False, True):
            say("case", what, lt, np.dtype(dtype).name, "columns", N, accumulate)
            C = dev(C0)
            sp.sp_matmul(A, dev(B), C, accumulate=accumulate)
            base = C0 if accumulate else np.zeros_like(C0)
            assert_product_close(C, ref + base, mag + np.abs(base), dtype, what)


@pytest.mark.parametrize("dtype,widths", [(np.float64, (2, 4, 8, 16, 32, 64, 128)), (np.float32, (4, 8, 16, 32, 64, 128, 256))])
@pytest.mark.parametrize("length", [55, 56, 95, 96, 447, 448])
def test_even_rows(dtype, widths, length):
    lens = np.full(9000 // length, length)
    lens[lens.size // 2] = min(4 * length - 4, 1500)         # still even: four times the mean at most
    check(lens, 1500, dtype, widths, "rows of %d" % length)


@pytest.mark.parametrize("lt", [(0, 1), (1, 1)])
def test_even_rows_among_empty_ones(lt):
    lens = np.full(150, 100)
    lens[::3] = 0
    lens[-1] = 0
    check(lens, 400, np.float64, (2, 32, 33), "rows of 100 among empty ones", lt)


@pytest.mark.parametrize("dtype,widths", [(np.float64, (2, 3, 7, 16, 33, 128, 131)), (np.float32, (2, 3, 4, 5, 8, 15, 32, 255, 260))])
@pytest.mark.parametrize("lens", [[1024] * 4, [1023, 1025, 2048, 0, 1, 3000], [0, 5000, 0, 0, 1, 5000, 0], [10240]])
def test_rows_that_fill_windows(dtype, widths, lens):
    check(lens, 10240, dtype, widths, "rows of " + str(lens))


@pytest.mark.parametrize("dtype,widths", [(np.float64, (2, 8, 33)), (np.float32, (3, 32))])
def test_rows_that_cross_more_than_64_windows(dtype, widths):
    """The carries of 65 and of 130 windows in one row, and a row of one window between them."""
    lens = np.concatenate([[66 * 1024 + 7], np.full(40, 3), [700, 131 * 1024 + 1], np.full(3000, 2)])
    check(lens, 140000, dtype, widths, "rows of 67,591 and 134,145")
