"""MTTKRP's padded copies of a factor matrix: made where gathers outnumber the rows, in 16-byte pieces or element by element, and
not where a long mode has few entries (the copy would be most of the work, and stay with the tensor).  Against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_04305_amd as sp
from gen import prng
from gpu_util import say, dev, gpu_pack, assert_product_close, DEV

pytestmark = pytest.mark.gpu
SEED = 20220308


def tensor(shape, nnz, dtype):
    lin = np.unique(prng.below(SEED, 1, nnz, int(np.prod(shape))).astype(np.int64))
    i, rest = lin // (shape[1] * shape[2]), lin % (shape[1] * shape[2])
    return [i, rest // shape[2], rest % shape[2]], prng.uniform_pm1(SEED, 2, lin.size, dtype=dtype)


@pytest.mark.parametrize("dtype,J,extra,copied", [(np.float64, 42, 0, True), (np.float64, 43, 0, True), (np.float64, 42, 3, True), (np.float32, 60, 0, True),
                                                  (np.float32, 61, 2, True), (np.float64, 48, 0, False), (np.float64, 33, 0, False)])
def test_large_factor(dtype, J, extra, copied):
    shape = (40, 30, 45000)
    coords, vals = tensor(shape, 2_200_000, dtype)
    T = gpu_pack((0, 1, 1), (0, 1, 2), shape, coords, vals)
    C = prng.uniform_pm1(SEED, 3, shape[1] * J, dtype=dtype).reshape(-1, J)
    D = prng.uniform_pm1(SEED, 4, shape[2] * J, dtype=dtype).reshape(-1, J)
    ref, mag = oracle.mttkrp_coo(shape, *coords, vals, C, D)
    wide = torch.full((shape[2], J + extra), float("nan"), dtype=T.dtype, device=DEV)
    wide[:, :J].copy_(dev(D))
    say("case large factor", np.dtype(dtype).name, J, "leading dimension", J + extra)
    before = sp.sp_tensor_info(T).derivedBytes
    A = sp.sp_mttkrp(T, dev(C), wide[:, :J])
    assert_product_close(A, ref, mag, dtype, "mttkrp")
    padded = shape[2] * ((J * np.dtype(dtype).itemsize + 127) // 128 * 128)
    assert (sp.sp_tensor_info(T).derivedBytes - before >= padded) == copied


@pytest.mark.parametrize("order", [(0, 1, 2), (0, 2, 1)])
@pytest.mark.parametrize("J", [33, 42])
def test_a_long_mode_with_few_entries_is_not_copied(order, J):
    shape = (50, 20, 600_000)
    coords, vals = tensor(shape, 30_000, np.float64)
    T = gpu_pack((0, 1, 1), order, shape, coords, vals)
    C, D = prng.uniform_pm1(SEED, 3, shape[1] * J).reshape(-1, J), prng.uniform_pm1(SEED, 4, shape[2] * J).reshape(-1, J)
    ref, mag = oracle.mttkrp_coo(shape, *coords, vals, C, D)
    A = sp.sp_mttkrp(T, dev(C), dev(D))
    assert_product_close(A, ref, mag, np.float64, "mttkrp")
    assert sp.sp_tensor_info(T).derivedBytes < 4 << 20
