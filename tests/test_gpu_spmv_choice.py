"""Which kernel a matrix-times-vector product runs when the library chooses, and what choosing costs, against the CPU checker: products
without sp_prepare before them keep to the packed storage where a regrouped copy would not pay, and can be recorded."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_04305_amd as sp
from paper_2202_04305_amd import binding
from gen import prng
from gpu_util import say, dev, assert_product_close, DEV

pytestmark = pytest.mark.gpu
SEED = 660203


def scattered(m, n, nnz, dtype=np.float64, stored=None):
    """About nnz entries anywhere in the first `stored` rows (all)."""
    lin = np.unique(prng.below(SEED + nnz, 1, nnz, (stored or m) * n))
    return [lin // n, lin % n], prng.uniform_pm1(SEED, 3, lin.size, dtype)


@pytest.mark.parametrize("lt,m,stored,n,nnz", [((0, 1), 100000, None, 3000000, 1500000), ((1, 1), 90000, 84000, 8000000, 2700000),
                                               ((1, 1), 100000, None, 3000000, 1500000), ((0, 1), 1000000, 90000, 3000000, 1500000)])
def test_product_without_prepare_reads_the_packed_storage(lt, m, stored, n, nnz):
    """1 to 2 M entries, or few row blocks: nothing is allocated and nothing is asked of the device; sp_prepare still gets the copy."""
    (rows, cols), vals = scattered(m, n, nnz, stored=stored)
    x = prng.uniform_pm1(SEED, 4, n, np.float64)
    ref, mag = oracle.matmul_coo((m, n), rows, cols, vals, x[:, None])
    alloc = binding._TorchAllocator(DEV)
    A = sp.sp_pack(sp.sp_encode(lt, (0, 1), 32, 32), (m, n), [dev(rows), dev(cols)], dev(vals), allocator=alloc)
    held = set(alloc.live)
    xd, y = dev(x), torch.full((m,), float("nan"), dtype=torch.float64, device=DEV)
    sp.sp_matmul(A, xd, y)
    info = sp.sp_tensor_info(A)
    say("case", lt, m, n, nnz, "kernel", info.spmvKernel)
    assert info.spmvKernel == 2 and info.lazyPrepares == 1 and set(alloc.live) == held
    assert_product_close(y[:, None], ref, mag, np.float64, "without sp_prepare")
    sp.sp_prepare(A, 1)
    assert sp.sp_tensor_info(A).spmvKernel == 4 and len(alloc.live) > len(held)
    y.fill_(float("nan"))
    sp.sp_matmul(A, xd, y)
    assert sp.sp_tensor_info(A).lazyPrepares == 1
    assert_product_close(y[:, None], ref, mag, np.float64, "after sp_prepare")


def test_product_of_a_middle_sized_matrix_can_be_recorded_without_prepare():
    m, n, nnz = 100000, 3000000, 1500000
    (rows, cols), vals = scattered(m, n, nnz)
    x = prng.uniform_pm1(SEED, 4, n, np.float64)
    ref, mag = oracle.matmul_coo((m, n), rows, cols, vals, x[:, None])
    A = sp.sp_pack(sp.sp_encode((0, 1), (0, 1), 32, 32), (m, n), [dev(rows), dev(cols)], dev(vals))
    xd, y = dev(x), torch.empty(m, dtype=torch.float64, device=DEV)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sp.sp_matmul(A, xd, y)
    for replay in range(3):
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert_product_close(y[:, None], ref, mag, np.float64, "replay %d" % replay)


def by_length(m, n, nnz, longest):
    """About nnz entries in rows sorted by length."""
    w = np.arange(1, m + 1, dtype=np.float64) ** -0.7
    lo, hi = 0.0, float(nnz)
    for _ in range(60):
        c = 0.5 * (lo + hi)
        lo, hi = (c, hi) if np.minimum(w * c, longest).round().sum() < nnz else (lo, c)
    lens = np.minimum(w * hi, longest).round().astype(np.int64)
    rows = np.repeat(np.arange(m), lens)
    lin = np.unique(rows * n + prng.below(SEED + longest, 5, rows.size, n))
    return lin // n, lin % n


def evenly(m, n, nnz):
    return scattered(m, n, nnz)[0]


def one_long(m, n, nnz, longest):
    (rows, cols), _ = scattered(m, n, nnz - longest)
    keep = rows != 17
    return (np.concatenate([rows[keep], np.full(longest, 17)]),
            np.concatenate([cols[keep], np.sort(prng.permutation(SEED, 6, n)[:longest])]))


@pytest.mark.parametrize("dtype,make,args,kernels", [
    (np.float32, one_long, (200000, 2000000, 3000000, 990000), (2,)),        # binned: 1256 us, streamed: 162
    (np.float32, by_length, (200000, 2000000, 3000000, 20000), (2,)),        # 131 and 39
    (np.float32, by_length, (200000, 2000000, 3000000, 64), (4,)),           # 26 and 38
    (np.float32, one_long, (200000, 2000000, 3000000, 3000), (4,)),          # 19 and 38
    (np.float64, by_length, (600000, 600000, 4500000, 5000), (2, 3)),        # row blocks of 2048 and 32 entries a bucket, one far above the mean
    (np.float64, evenly, (525000, 420000, 6000000), (4,)),                   # the same with an x of 3.4 MB and no block above the mean
])
def test_the_choice_looks_at_the_heaviest_row_block(dtype, make, args, kernels):
    m, n = args[:2]
    rows, cols = make(*args)
    vals, x = prng.uniform_pm1(SEED, 7, rows.size, dtype), prng.uniform_pm1(SEED, 8, n, dtype)
    ref, mag = oracle.matmul_coo((m, n), rows, cols, vals, x[:, None])
    A = sp.sp_pack(sp.sp_encode((0, 1), (0, 1), 32, 32), (m, n), [dev(rows), dev(cols)], dev(vals))
    sp.sp_prepare(A, 1)
    info = sp.sp_tensor_info(A)
    say("case", np.dtype(dtype).name, make.__name__, args, "longest row", info.maxSegment, "kernel", info.spmvKernel)
    assert info.spmvKernel in kernels
    y = torch.full((m,), float("nan"), dtype=torch.float32 if dtype == np.float32 else torch.float64, device=DEV)
    sp.sp_matmul(A, dev(x), y)
    assert_product_close(y[:, None], ref, mag, dtype, make.__name__)
