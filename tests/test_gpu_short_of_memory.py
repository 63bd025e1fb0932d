"""What the library does when an allocator refuses a block that a slower path can do without: the slower path runs, and nothing that
the refused request left behind (HIP keeps the error of a failed hipMalloc for the next question) is taken for its failure."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2202_04305_amd as sp
from paper_2202_04305_amd import binding
from gen import prng
from gpu_util import say, dev, assert_product_close, assert_storage_equal, DEV

pytestmark = pytest.mark.gpu
SEED = 430917


def hip_runtime():
    """The HIP runtime that this process has loaded."""
    path = {line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line}
    return ctypes.CDLL(path.pop())


class PickyAllocator(binding._TorchAllocator):
    """torch's allocator behind the callbacks; a request that `refuses(bytes)` fails as hipMalloc fails."""

    def __init__(self, refuses=lambda nbytes: False):
        super().__init__(DEV)
        self.refuses, self.sizes, self.refused = refuses, [], 0
        self.hip = hip_runtime()

    def _alloc(self, nbytes, ctx):
        self.sizes.append(nbytes)
        if self.refuses(nbytes):
            p = ctypes.c_void_p()
            assert self.hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 60)) != 0        # more than any GPU has
            self.refused += 1
            return None
        return super()._alloc(nbytes, ctx)


def entries(m, n, nnz, dtype):
    lin = np.unique(prng.below(SEED, 1, nnz * 2, m * n))
    lin = lin[prng.permutation(SEED, 2, lin.size)][:nnz]
    return [lin // n, lin % n], prng.uniform_pm1(SEED, 3, nnz, dtype)


@pytest.mark.parametrize("fmt", [((0, 1), (0, 1)), ((1, 1), (0, 1)), ((1, 0), (0, 1))])
@pytest.mark.parametrize("nnz", [50000, 1300000])
def test_no_room_for_the_buckets(fmt, nnz):
    """The sort by buckets takes its scratch as one block; without it the stable sorts build the same storage."""
    shape = (60000, 50)
    coords, vals = entries(*shape, nnz, np.float64)
    ref = oracle.pack(*fmt, shape, coords, vals, 32, 32)
    enc, cd, vd = sp.sp_encode(*fmt, 32, 32), [dev(c) for c in coords], dev(vals)
    asked = []
    for mode in (0, 1):
        alloc = PickyAllocator()
        sp.sp_pack_sort_mode(mode)
        try:
            sp.sp_pack(enc, shape, cd, vd, allocator=alloc).free()
        finally:
            sp.sp_pack_sort_mode(0)
        asked.append(alloc.sizes)
    block = max(set(asked[0]) - set(asked[1]))
    say("case", fmt, nnz, "block of the buckets", block)
    assert block > 24 * nnz
    alloc = PickyAllocator(lambda nbytes: nbytes == block)
    A = sp.sp_pack(enc, shape, cd, vd, allocator=alloc)
    assert alloc.refused == 1
    assert_storage_equal(A, ref)
    A.free()
    assert not alloc.live


@pytest.mark.parametrize("lt", [(0, 1), (1, 1)])
@pytest.mark.parametrize("m,n,nnz", [(100000, 3000000, 1500000), (600000, 600000, 5000000)])
def test_no_room_for_the_copy_of_a_matrix_times_vector(lt, m, n, nnz):
    """Scattered columns: the automatic choice is a kernel over a regrouped copy.  Without room for it the streamed kernel, which needs
    none, computes the product; a kernel that was asked for still is an error."""
    (rows, cols), vals = entries(m, n, nnz, np.float64)
    x = prng.uniform_pm1(SEED, 4, n, np.float64)
    ref, mag = oracle.matmul_coo((m, n), rows, cols, vals, x[:, None])
    enc, cd, vd, xd = sp.sp_encode(lt, (0, 1), 32, 32), [dev(rows), dev(cols)], dev(vals), dev(x)
    y = torch.empty(m, dtype=torch.float64, device=DEV)
    A = sp.sp_pack(enc, (m, n), cd, vd)
    sp.sp_prepare(A, 1)
    assert sp.sp_tensor_info(A).spmvKernel == 4
    for prepared in (True, False):
        alloc = PickyAllocator()
        A = sp.sp_pack(enc, (m, n), cd, vd, allocator=alloc)
        held = set(alloc.live)
        alloc.refuses = lambda nbytes: nbytes > 4096
        if prepared:
            sp.sp_prepare(A, 1)
        sp.sp_matmul(A, xd, y)
        say("case", lt, (m, n, nnz), "prepared" if prepared else "not prepared", "refused", alloc.refused)
        assert sp.sp_tensor_info(A).spmvKernel == 2 and set(alloc.live) == held
        if prepared:
            assert alloc.refused >= 1
        assert_product_close(y[:, None], ref, mag, np.float64, "without the copy")
        sp.sp_tensor_tune(A, sp.SP_TUNE_SPMV_KERNEL, 4)
        with pytest.raises(sp.SpError) as e:
            sp.sp_prepare(A, 1)
        assert e.value.code == 12
        A.free()
        assert not alloc.live
