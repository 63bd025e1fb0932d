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
