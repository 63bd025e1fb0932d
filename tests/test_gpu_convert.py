"""sp_convert against the CPU checker: the storage of the target encoding bit for bit, whatever the source's.

Sizes: one entry, the edges of the 4096-position tiles, a source whose tile spans more rows than the LDS holds; ranks two and
three, dense levels above and below compressed ones (their zeros become stored entries), every pair of index widths.
"""
import numpy as np
import pytest

import oracle
import paper_2202_04305_amd as sp
from gen import workloads as W, prng
from gpu_util import say, dev, gpu_pack, assert_storage_equal

pytestmark = pytest.mark.gpu


def check(shape, coords, vals, src, dst, widths_src=(32, 32), widths_dst=(32, 32)):
    say("case convert", shape, len(vals), src, dst, widths_src, widths_dst)
    A = gpu_pack(src[0], src[1], shape, coords, vals, *widths_src)
    T = sp.sp_convert(A, sp.sp_encode(dst[0], dst[1], *widths_dst))
    mid = oracle.pack(src[0], src[1], shape, coords, vals, *widths_src)
    c2, v2 = mid.unpack()                                   # every stored position, zeros under dense levels included
    assert_storage_equal(T, oracle.pack(dst[0], dst[1], shape, c2, v2.astype(vals.dtype), *widths_dst))


CSR, CSC, DCSR, CD, DD = ((0, 1), (0, 1)), ((0, 1), (1, 0)), ((1, 1), (0, 1)), ((1, 0), (0, 1)), ((0, 0), (1, 0))


@pytest.mark.parametrize("nnz", [1, 2, 4095, 4096, 4097, 12289])
@pytest.mark.parametrize("src,dst", [(CSR, CSC), (CSC, CSR), (DCSR, CSC), (CSR, DCSR)])
def test_convert_tile_edges(nnz, src, dst):
    w = W.uniform_random(300, 257, nnz)
    check(w.shape, [w.rows, w.cols], w.vals, src, dst)


@pytest.mark.parametrize("src", [CSR, DCSR, CSC])
def test_convert_more_rows_in_a_tile_than_the_lds_holds(src):
    w = W.uniform_random(40000, 50000, 6000)
    check(w.shape, [w.rows, w.cols], w.vals, src, CSC if src is not CSC else CSR)


@pytest.mark.parametrize("src", [CD, DD])
@pytest.mark.parametrize("dst", [CSR, CSC, DCSR])
def test_convert_from_dense_levels(src, dst):
    w = W.uniform_random(90, 110, 500)
    check(w.shape, [w.rows, w.cols], w.vals, src, dst)


@pytest.mark.parametrize("widths", [((32, 64), (64, 32)), ((64, 32), (32, 64)), ((64, 64), (16, 16)), ((16, 16), (64, 64))])
def test_convert_widths(widths):
    w = W.uniform_random(200, 300, 5000)
    w.vals = w.vals.astype(np.float32)
    check(w.shape, [w.rows, w.cols], w.vals, CSR, CSC, *widths)


@pytest.mark.parametrize("order", [(0, 2, 1), (2, 0, 1), (1, 2, 0)])
@pytest.mark.parametrize("lt", [(1, 1, 1), (0, 1, 1), (1, 0, 1), (1, 1, 0)])
def test_convert_rank_three(lt, order):
    rng = np.random.default_rng(3)
    shape = (13, 17, 60)
    keys = rng.choice(13 * 17 * 60, 4500, replace=False)
    coords = [keys // (17 * 60), keys // 60 % 17, keys % 60]
    vals = rng.standard_normal(4500)
    check(shape, coords, vals, ((1, 1, 1), (0, 1, 2)), (lt, order))
    check(shape, coords, vals, (lt, order), ((1, 1, 1), (0, 1, 2)))


@pytest.mark.parametrize("per_row", [64, 128])
@pytest.mark.parametrize("full", ["first", "last"])
def test_a_full_column_at_the_same_place_of_every_row(per_row, full):
    """Rows of 64 or 128 entries, one column in all of them: whatever places of a row the sort's sample looks at, the columns come out
    in order (a column of 20,000 entries fits no block of the sort by buckets, nor of the most-significant-digit-first one)."""
    m, n = 20000, 1 << 16
    r = np.repeat(np.arange(m, dtype=np.int64), per_row)
    c = np.tile(np.arange(per_row, dtype=np.int64), m) * (n // per_row - 3) + r % 700
    c[(per_row - 1 if full == "last" else 0)::per_row] = n - 1 if full == "last" else 0
    if full == "first":
        c[1::per_row] = np.maximum(c[1::per_row], 1)
    v = prng.uniform_pm1(W.BASE_SEED, 77, r.size)
    A = gpu_pack((0, 1), (0, 1), (m, n), [r, c], v)
    say("case full column", full, "rows of", per_row)
    B = sp.sp_convert(A, sp.sp_encode((0, 1), (1, 0), 32, 32))
    assert_storage_equal(B, oracle.pack((0, 1), (1, 0), (m, n), [r, c], v, 32, 32))
