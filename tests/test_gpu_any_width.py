"""Dense operands of any width, leading dimension and element-aligned address, against the CPU checker.

The kernels load 16 bytes wherever a row begins and move the last load of a row back to the row's end, so the sizes are
the edges of that rule: fewer columns than a load holds, one more and one less than a whole number of loads; rows longer
than a window of 1024 stored entries; an infinity in the columns that two loads share.  Most inputs are of a few windows, and
few windows share the columns out four loads to a block; the tests "of many windows" have more than 512, so that a row of
the operand takes 33 to 64 lanes, one more than a wave covers, and a second tile of columns.
Tolerance: the products' own, 1e-12 (f64) / 1e-5 (f32) times sum|a*b| per element.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_04305_amd as sp
from gen import workloads as W, prng
from gpu_util import say, dev, gpu_pack, assert_product_close, DEV

pytestmark = pytest.mark.gpu


def embedded(a, ld, offset):
    """The array as a window of a wider one that begins `offset` elements past a 256-byte boundary, NaN around it."""
    rows, cols = a.shape
    flat = torch.full((offset + rows * ld + 64,), float("nan"), dtype=torch.from_numpy(a[:1]).dtype, device=DEV)
    view = flat[offset:offset + rows * ld].view(rows, ld)[:, :cols]
    view.copy_(dev(a))
    return flat, view


@pytest.mark.parametrize("lt", [(0, 1), (1, 1)])
@pytest.mark.parametrize("dtype,N", [(np.float64, n) for n in (2, 3, 5, 33, 64, 127, 129, 131)] +
                         [(np.float32, n) for n in (2, 3, 4, 5, 7, 33, 64, 255, 257)])
def test_spmm_any_width_and_address(lt, dtype, N):
    w = W.cfg2_powerlaw_csr(700, 3000, mean=40.0, sigma=1.5, cap=2900)
    w.rows = w.rows * 2                                    # an empty row after every row
    w.shape = (1400, 3000)
    vals = w.vals.astype(dtype)
    A = gpu_pack(lt, (0, 1), w.shape, [w.rows, w.cols], vals)
    B = prng.uniform_pm1(7, 1, w.shape[1] * N, dtype=dtype).reshape(-1, N)
    C0 = prng.uniform_pm1(7, 2, w.shape[0] * N, dtype=dtype).reshape(-1, N)
    ref, mag = oracle.matmul_coo(w.shape, w.rows, w.cols, vals, B)
    for extra, offset in [(0, 0), (1, 1), (3, 2)]:
        for accumulate in (False, True):
            say("case spmm any width", lt, dtype.__name__, N, extra, offset, accumulate)
            _, Bd = embedded(B, N + extra, offset)
            flat, Cd = embedded(C0, N + extra, offset)
            before = flat.clone()
            sp.sp_matmul(A, Bd, Cd, accumulate=accumulate)
            base = C0 if accumulate else np.zeros_like(C0)
            assert_product_close(Cd, ref + base, mag + np.abs(base), dtype, "spmm")
            written = torch.zeros_like(flat, dtype=torch.bool)
            written[offset:offset + w.shape[0] * (N + extra)].view(w.shape[0], N + extra)[:, :N] = True
            assert torch.equal(torch.isnan(flat[~written]), torch.isnan(before[~written]))


@pytest.mark.parametrize("N", [3, 33])
def test_spmm_any_width_recorded_before_any_scratch_exists(N):
    """Under capture, on a tensor that was never prepared, the product takes the kernel that needs no scratch."""
    w = W.cfg2_powerlaw_csr(3000, 2500, cap=900)
    enc = sp.sp_encode((0, 1), (0, 1), 32, 32)
    A = sp.sp_pack(enc, w.shape, [dev(w.rows), dev(w.cols)], dev(w.vals))
    B = prng.uniform_pm1(7, 3, w.shape[1] * N).reshape(-1, N)
    ref, mag = oracle.matmul_coo(w.shape, w.rows, w.cols, w.vals, B)
    Bd, Cd = dev(B), torch.empty((w.shape[0], N), dtype=torch.float64, device=DEV)
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):                 # never prepared: nothing may be allocated here
        sp.sp_matmul(A, Bd, Cd)
    for _ in range(3):
        Cd.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert_product_close(Cd, ref, mag, np.float64, "replay")


@pytest.mark.parametrize("dtype,K", [(np.float64, k) for k in (2, 3, 15, 17, 33, 64, 127, 129)] +
                         [(np.float32, k) for k in (3, 4, 5, 31, 33, 64, 255, 257)])
def test_sddmm_any_width_and_address(dtype, K):
    """Rows longer than a window, empty rows, operands inside wider ones; CSR and DCSR."""
    w = W.cfg2_powerlaw_csr(700, 3000, mean=40.0, sigma=1.5, cap=2900)
    w.rows = w.rows * 2
    w.shape = (1400, 3000)
    vals = w.vals.astype(dtype)
    A = prng.uniform_pm1(8, 1, w.shape[0] * K, dtype=dtype).reshape(-1, K)
    B = prng.uniform_pm1(8, 2, w.shape[1] * K, dtype=dtype).reshape(-1, K)
    x, mag = oracle.sddmm_coo(w.shape, w.rows, w.cols, vals, A, np.ascontiguousarray(B.T))
    for lt in [(0, 1), (1, 1)]:
        S = gpu_pack(lt, (0, 1), w.shape, [w.rows, w.cols], vals)
        xs = oracle.pack(lt, (0, 1), w.shape, [w.rows, w.cols], x, 32, 32).values
        ms = oracle.pack(lt, (0, 1), w.shape, [w.rows, w.cols], mag, 32, 32).values
        for extra, offset in [(0, 0), (1, 1), (3, 2)]:
            say("case sddmm any width", lt, dtype.__name__, K, extra, offset)
            Ad, Bd = embedded(A, K + extra, offset)[1], embedded(B, K + extra, offset)[1]
            X = torch.full((w.nnz,), float("nan"), dtype=S.dtype, device=DEV)
            sp.sp_sddmm(S, Ad, Bd, X, b_is_transposed=True)
            assert_product_close(X, xs, ms, dtype, "sddmm")


@pytest.mark.parametrize("K", [5, 33])
def test_sddmm_keeps_infinities_where_two_loads_meet(K):
    """inf * 0 in a column that two loads cover must not turn a row's infinite sum into NaN, nor spread to other rows."""
    w = W.uniform_random(60, 50, 900)
    A, B = np.ones((60, K)), np.ones((50, K))
    B[7, K - 2] = B[9, K - 1] = np.inf
    S = gpu_pack((0, 1), (0, 1), w.shape, [w.rows, w.cols], np.ones(w.nnz))
    X = sp.sp_sddmm(S, dev(A), dev(B), b_is_transposed=True).cpu().numpy()
    hit = np.isin(sp.sp_crd(S, 1).cpu().numpy(), (7, 9))
    assert hit.any() and np.all(np.isposinf(X[hit])) and np.all(X[~hit] == K)


@pytest.mark.parametrize("order", [(0, 1, 2), (0, 2, 1)])
@pytest.mark.parametrize("dtype,J", [(np.float64, j) for j in (2, 3, 33, 127, 129)] + [(np.float32, j) for j in (2, 3, 5, 42, 255, 257)])
def test_mttkrp_any_width_and_address(order, dtype, J):
    w = W.tensor3_slices(I=40, K=90, L=200, nnz=9000, k_mean=25, l_mean=60, sigma=1.2, J=J, dtype=dtype)
    C, D = w.factors()
    ref, mag = oracle.mttkrp_coo(w.shape, w.ci, w.ck, w.cl, w.vals, C, D)
    T = gpu_pack((0, 1, 1), order, w.shape, [w.ci, w.ck, w.cl], w.vals)
    A0 = prng.uniform_pm1(9, 1, w.shape[0] * J, dtype=dtype).reshape(-1, J)
    for extra, offset, accumulate in [(0, 0, False), (1, 1, False), (3, 2, True)]:
        say("case mttkrp any width", order, dtype.__name__, J, extra, offset)
        Cd, Dd = embedded(C, J + extra, offset)[1], embedded(D, J + extra, offset)[1]
        flat, Ad = embedded(A0, J + extra, offset)
        before = flat.clone()
        sp.sp_mttkrp(T, Cd, Dd, A=Ad, accumulate=accumulate)
        base = A0 if accumulate else np.zeros_like(A0)
        assert_product_close(Ad, ref + base, mag + np.abs(base), dtype, "mttkrp")
        written = torch.zeros_like(flat, dtype=torch.bool)
        written[offset:offset + w.shape[0] * (J + extra)].view(w.shape[0], J + extra)[:, :J] = True
        assert torch.equal(torch.isnan(flat[~written]), torch.isnan(before[~written]))


@pytest.fixture(scope="module")
def many_windows():
    w = W.cfg2_powerlaw_csr(20000, 4000, mean=30.0, sigma=1.3, cap=3500)
    assert w.nnz > 512 * 1024
    return w


@pytest.mark.parametrize("dtype,N", [(np.float64, n) for n in (67, 127, 129, 131)] + [(np.float32, n) for n in (255, 257)])
def test_spmm_of_many_windows(many_windows, dtype, N):
    w = many_windows
    vals = w.vals.astype(dtype)
    A = gpu_pack((0, 1), (0, 1), w.shape, [w.rows, w.cols], vals)
    B = prng.uniform_pm1(7, 1, w.shape[1] * N, dtype=dtype).reshape(-1, N)
    ref, mag = oracle.matmul_coo(w.shape, w.rows, w.cols, vals, B)
    for extra, offset in [(0, 0), (1, 1)]:
        say("case spmm many windows", dtype.__name__, N, extra, offset)
        _, Bd = embedded(B, N + extra, offset)
        _, Cd = embedded(np.zeros((w.shape[0], N), dtype=dtype), N + extra, offset)
        sp.sp_matmul(A, Bd, Cd)
        assert_product_close(Cd, ref, mag, dtype, "spmm")


@pytest.mark.parametrize("dtype,J", [(np.float64, j) for j in (67, 127, 129)] + [(np.float32, j) for j in (255, 257)])
def test_mttkrp_of_many_windows(dtype, J):
    w = W.tensor3_slices(I=300, K=200, L=500, nnz=600000, k_mean=80, l_mean=120, sigma=0.8, J=J, dtype=dtype)
    C, D = w.factors()
    ref, mag = oracle.mttkrp_coo(w.shape, w.ci, w.ck, w.cl, w.vals, C, D)
    T = gpu_pack((0, 1, 1), (0, 1, 2), w.shape, [w.ci, w.ck, w.cl], w.vals)
    assert len(w.vals) > 512 * 1024
    for extra, offset in [(0, 0), (1, 1)]:
        say("case mttkrp many windows", dtype.__name__, J, extra, offset)
        Cd, Dd = embedded(C, J + extra, offset)[1], embedded(D, J + extra, offset)[1]
        assert_product_close(sp.sp_mttkrp(T, Cd, Dd), ref, mag, dtype, "mttkrp")


@pytest.mark.parametrize("dtype,K", [(np.float64, k) for k in (5, 33, 64, 100)] + [(np.float32, k) for k in (5, 33, 64, 100, 200)])
def test_sddmm_of_many_windows(dtype, K):
    """More than 1024 windows: a block takes a whole one.  Small whole numbers, so that every sum is exact: bit for bit."""
    w = W.cfg2_powerlaw_csr(40000, 5000, mean=36.0, sigma=1.2, cap=3000)
    assert w.nnz > 1024 * 1024
    vals = (1 + prng.below(8, 3, w.nnz, 3)).astype(dtype)
    A = (prng.below(8, 1, w.shape[0] * K, 7).astype(dtype) - 3).reshape(-1, K)
    B = (prng.below(8, 2, w.shape[1] * K, 7).astype(dtype) - 3).reshape(-1, K)
    S = gpu_pack((0, 1), (0, 1), w.shape, [w.rows, w.cols], vals)
    say("case sddmm many windows", dtype.__name__, K)
    X = sp.sp_sddmm(S, dev(A), dev(B), b_is_transposed=True)
    co, v = sp.sp_unpack(S)
    exact = torch.cat([v[e:e + (1 << 17)] * (dev(A)[co[0][e:e + (1 << 17)]] * dev(B)[co[1][e:e + (1 << 17)]]).sum(1)
                       for e in range(0, w.nnz, 1 << 17)])
    assert torch.equal(X, exact)
