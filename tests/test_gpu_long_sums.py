"""Long sums lose no more than their first few terms: one large term and many that a sum as large as it rounds away.

The large term is 1, the others 0.45 of the last place of 1, so a plain chain of n terms is off by 0.9 n u (u: half of that last
place, the unit roundoff).  Bounds count the roundings a term can pass through: each is at most u times the sum so far."""
import numpy as np
import pytest
import torch

import paper_2202_04305_amd as sp
from gen import prng
from gpu_util import say, dev, gpu_pack, DEV

pytestmark = pytest.mark.gpu


def unit(dtype):
    return float(np.finfo(dtype).eps) / 2


def rows_with_one_large_entry(dtype, long_rows, length, short_rows):
    """rows, cols, values, and every row's exact sum (in long double): long rows among short ones, so that neither is even."""
    lens = np.full(long_rows + short_rows, 3, dtype=np.int64)
    lens[prng.permutation(3, 1, lens.size)[:long_rows]] = length
    rows = np.repeat(np.arange(lens.size, dtype=np.int64), lens)
    first = np.cumsum(lens) - lens
    cols = np.arange(rows.size, dtype=np.int64) - np.repeat(first, lens)
    vals = np.full(rows.size, 0.9 * unit(dtype), dtype=dtype)
    vals[first] = 1
    exact = 1 + (lens - 1).astype(np.longdouble) * np.longdouble(vals[1])
    return rows, cols, vals, lens, exact


def worst(got, exact, dtype):
    """largest error of any element, in units of u times the row's sum of magnitudes"""
    err = np.abs(got.cpu().numpy().astype(np.longdouble) - exact.reshape(-1, 1))
    return float((err / exact.reshape(-1, 1)).max() / unit(dtype))


@pytest.mark.parametrize("lt", [(0, 1), (1, 1)])
@pytest.mark.parametrize("dtype,N", [(np.float64, n) for n in (2, 8, 33, 64, 128)] + [(np.float32, n) for n in (3, 8, 32, 65, 256)])
def test_spmm(lt, dtype, N):
    """More than 512 windows, so that a row of B gets all the lanes it needs and a group up to 256 entries.
    Four entries in a chain, the long sum's rounding, up to eight levels among the groups of a window, one more for a window that
    the row crosses: 14."""
    rows, cols, vals, lens, exact = rows_with_one_large_entry(dtype, 450, 1000, 40000)
    A = gpu_pack(lt, (0, 1), (lens.size, 1000), [rows, cols], vals)
    B = torch.ones((1000, N), dtype=A.dtype, device=DEV)
    C = torch.full((lens.size, N), float("nan"), dtype=A.dtype, device=DEV)
    sp.sp_matmul(A, B, C)
    say("case spmm long sums", lt, dtype.__name__, N, "worst", worst(C, exact, dtype))
    assert worst(C, exact, dtype) <= 14


@pytest.mark.parametrize("dtype,N", [(np.float64, 8), (np.float64, 33), (np.float32, 32), (np.float32, 3)])
def test_spmm_keeps_infinities_and_nan(dtype, N):
    """An infinite product gives an infinite sum whatever is added after it; a NaN gives NaN; neither reaches another row or column."""
    rows, cols, vals, lens, _ = rows_with_one_large_entry(dtype, 20, 700, 2000)
    A = gpu_pack((0, 1), (0, 1), (lens.size, 700), [rows, cols], vals)
    B = np.ones((700, N), dtype=dtype)
    B[5, 0], B[9, N - 1] = np.inf, np.nan
    C = sp.sp_matmul(A, dev(B), torch.empty((lens.size, N), dtype=A.dtype, device=DEV)).cpu().numpy()
    assert np.all(np.isposinf(C[lens > 5, 0])) and np.all(np.isnan(C[lens > 9, N - 1]))
    assert np.all(np.isfinite(C[:, 1:N - 1])) and np.all(np.isfinite(C[lens <= 5]))


@pytest.mark.parametrize("dtype,K", [(np.float64, k) for k in (16, 33, 64, 128)] + [(np.float32, k) for k in (16, 33, 100, 128, 256)])
def test_sddmm(dtype, K):
    """A dot product is a tree: a chain of the products of one 16-byte load, three levels among a lane's loads, three among its
    eight lanes, one multiplication: 4 + 3 + 3 + 1 = 11."""
    rows, cols, vals, lens, _ = rows_with_one_large_entry(dtype, 5, 300, 100)
    S = gpu_pack((0, 1), (0, 1), (lens.size, 300), [rows, cols], np.ones_like(vals))
    A, B = np.full((lens.size, K), 0.9 * unit(dtype), dtype=dtype), np.ones((300, K), dtype=dtype)
    A[:, 0] = 1
    exact = np.full(rows.size, 1 + (K - 1) * np.longdouble(A[0, 1]))
    X = sp.sp_sddmm(S, dev(A), dev(B), b_is_transposed=True)
    say("case sddmm long sums", dtype.__name__, K, "worst", worst(X.reshape(-1, 1), exact, dtype))
    assert worst(X.reshape(-1, 1), exact, dtype) <= 11


@pytest.mark.parametrize("fibres", ["one", "many"])
@pytest.mark.parametrize("dtype,J", [(np.float64, j) for j in (8, 42, 64, 127)] + [(np.float32, j) for j in (16, 42, 256)])
def test_mttkrp(fibres, dtype, J):
    """Slices of 900 entries, in one fibre or in as many, in more than 512 windows.
    Four entries in a chain, one multiplication by the fibre's row, eight such fours, eight of these in a run, one more where the two
    meet, up to eight levels among the groups of a window, three for the windows a slice crosses: 33."""
    slices, length = 640, 900
    i = np.repeat(np.arange(slices, dtype=np.int64), length)
    at = np.tile(np.arange(length, dtype=np.int64), slices)
    k, l = (np.zeros_like(at), at) if fibres == "one" else (at, at % 3)
    vals = np.full(i.size, 0.9 * unit(dtype), dtype=dtype)
    vals[at == 0] = 1
    T = gpu_pack((0, 1, 1), (0, 1, 2), (slices, length, length), [i, k, l], vals)
    ones = torch.ones((length, J), dtype=T.dtype, device=DEV)
    A = sp.sp_mttkrp(T, ones, ones)
    exact = np.full(slices, 1 + (length - 1) * np.longdouble(vals[1]))
    say("case mttkrp long sums", fibres, dtype.__name__, J, "worst", worst(A, exact, dtype))
    assert worst(A, exact, dtype) <= 33


def test_mttkrp_keeps_infinities():
    """A row of either factor that is infinite in one column: the slices that reach it are infinite there and nowhere else.  All
    other terms are positive, so nothing may turn into NaN, wherever a run of entries is cut."""
    slices, K, L, J = 300, 50, 40, 9
    p = prng.permutation(5, 1, slices * K * L)[:60000].astype(np.int64)
    p.sort()
    i, k, l = p // (K * L), p // L % K, p % L
    T = gpu_pack((0, 1, 1), (0, 1, 2), (slices, K, L), [i, k, l], np.ones(p.size))
    for which in (0, 1):
        C, D = np.ones((K, J)), np.ones((L, J))
        (C if which == 0 else D)[7, 4] = np.inf
        A = sp.sp_mttkrp(T, dev(C), dev(D)).cpu().numpy()
        hit = np.zeros(slices, dtype=bool)
        hit[i[(k if which == 0 else l) == 7]] = True
        assert hit.any() and np.all(np.isposinf(A[hit, 4])) and np.all(np.isfinite(np.delete(A, 4, axis=1))) and np.all(np.isfinite(A[~hit]))
