"""Matrix times vector where only some rows are stored, against the CPU checker: the streamed kernel, and the binned one, whose first
pass clears the other rows, at the edges of their windows of 1024 entries, row blocks and panels; rows that are not
stored stay untouched under accumulation."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_04305_amd as sp
from gen import prng
from gpu_util import say, dev, gpu_pack, assert_product_close, DEV

pytestmark = pytest.mark.gpu
SEED = 91177


def matrix(kind):
    """m, n, rows, columns: stored rows with gaps between them."""
    if kind == "one row":
        lens, ids, m, n = [700], [3], 9, 1000
    elif kind == "windows":                      # rows that begin and end where windows do, fill several, and share one
        lens, ids, m, n = [1024, 1024, 2048, 1, 1023, 3000, 100, 972, 1024, 5], [0, 1, 7, 50, 51, 52, 400, 4000, 4001, 70000], 70001, 5000
    elif kind == "first and last rows empty":
        lens, ids, m, n = [40] * 300, [1000 + 37 * i for i in range(300)], 30000, 20000
    else:                                        # more than one row block of 2048 and panel of 8192
        lens, ids, m, n = [32] * 5000, [3 * i + i // 7 for i in range(5000)], 20000, 30000
    rows = np.repeat(np.asarray(ids, np.int64), lens)
    cols = np.concatenate([np.sort(prng.permutation(SEED + i, 1, n)[:k]) for i, k in enumerate(lens)]).astype(np.int64)
    return m, n, rows, cols


@pytest.mark.parametrize("kernel", [2, 4])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("kind", ["one row", "windows", "first and last rows empty", "row blocks"])
def test_rows_that_are_not_stored(kind, dtype, kernel):
    m, n, rows, cols = matrix(kind)
    p = prng.permutation(SEED, 2, rows.size)
    vals = prng.uniform_pm1(SEED, 3, rows.size, dtype)
    x = prng.uniform_pm1(SEED, 4, n, dtype)
    ref, mag = oracle.matmul_coo((m, n), rows[p], cols[p], vals, x[:, None])
    for pw, cw in ((32, 32), (64, 64)):
        say("case", kind, dtype.__name__, "kernel", kernel, pw, cw)
        A = gpu_pack((1, 1), (0, 1), (m, n), [rows[p], cols[p]], vals, pw, cw)
        sp.sp_tensor_tune(A, sp.SP_TUNE_SPMV_KERNEL, kernel)
        sp.sp_prepare(A, 1)
        y = torch.full((m,), float("nan"), dtype=torch.float64 if dtype == np.float64 else torch.float32, device=DEV)
        for _ in range(2):
            sp.sp_matmul(A, dev(x), y)
            assert_product_close(y[:, None], ref, mag, dtype, kind)
        wide = torch.full((m, 3), 7.0, dtype=y.dtype, device=DEV)                # a column of a wider array: other columns stay
        sp.sp_matmul(A, dev(x), wide[:, 1], N=1, ldb=1, ldc=3)
        assert_product_close(wide[:, 1:2], ref, mag, dtype, kind + ", a strided result")
        assert bool((wide[:, 0] == 7).all()) and bool((wide[:, 2] == 7).all())
        z = torch.full((m,), 5.0, dtype=y.dtype, device=DEV)
        sp.sp_matmul(A, dev(x), z, accumulate=True)
        empty = torch.ones(m, dtype=torch.bool, device=DEV)
        empty[dev(np.unique(rows))] = False
        assert bool((z[empty] == 5).all())
        assert_product_close((z - 5.0)[:, None], ref, mag + 8.0, dtype, kind + ", accumulated")


def test_the_choice_keeps_rounding_of_long_rows():
    """f64 rows beyond 64 entries keep the kernels that add in trees at sizes where the binned copy would be faster."""
    m, n = 100000, 1 << 21
    nnz = 2200000
    lin = np.unique(prng.below(SEED, 7, int(nnz * 1.02), m * n))[:nnz - 300]
    long_row = np.arange(300, dtype=np.int64) * 5000 + 17 * n
    for extra, kernels in ((None, (4,)), (long_row, (2, 3))):
        keys = lin if extra is None else np.unique(np.concatenate([lin[lin // n != 17], extra]))
        A = gpu_pack((1, 1), (0, 1), (m, n), [keys // n, keys % n], np.ones(keys.size))
        sp.sp_prepare(A, 1)
        info = sp.sp_tensor_info(A)
        say("longest row", info.maxSegment, "kernel", info.spmvKernel)
        assert info.spmvKernel in kernels
        y = torch.full((m,), float("nan"), dtype=torch.float64, device=DEV)
        sp.sp_matmul(A, torch.ones(n, dtype=torch.float64, device=DEV), y)
        assert np.array_equal(y.cpu().numpy(), np.bincount(keys // n, minlength=m).astype(np.float64))
